"""K and V (and Q, dO of the backward) of a batch of one, read where the caller holds them at any Ulysses degree: bitwise
what the staged copies give, which tensors that do not lie on 16 bytes still take, and where items are whole, bitwise what the
all-to-alls and the ring loop give as calls of their own."""
import pytest
import torch

import paper_2405_07719_amd as usp

pytestmark = pytest.mark.gpu

# ..., how the launch divides the rank: whole items, V as rows / V in transposed tiles; heaviest tiles cut; every tile cut.
# A ring of two with a ragged last key tile, and tiles that end with a run, among them.
SHAPES = [(16384, 16, 4, 2, 1, 128, True, True, "whole"), (12288, 32, 8, 8, 1, 64, False, True, "whole"),
          (4 * 1100, 128, 16, 2, 2, 128, True, True, "whole"), (16384, 32, 2, 2, 1, 128, True, True, "whole, V in tiles"),
          (24576, 32, 8, 8, 1, 128, True, True, "heaviest cut"), (8192, 8, 4, 2, 1, 128, True, True, "heaviest cut"),
          (10240, 32, 8, 8, 1, 128, True, False, "heaviest cut"), (4 * 1100, 16, 8, 2, 2, 128, True, True, "all cut")]
# V staged as rows, which tensors that do not lie on 16 bytes can be (tiles are not made from such: refused)
ROWS_STAGED = {SHAPES[5], SHAPES[6], SHAPES[7]}


def shifted(t):
    """The same values at an address that is 2 bytes past a multiple of 16."""
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)
    out = buf[1:1 + t.numel()].view(t.shape)
    return out.copy_(t)


def dense_forward(p, q, k, v, rank):
    """The rank's O and LSE through the separate entry points: all-to-alls to tensors in head layout, its ring loop in one launch."""
    bs, L, U, R, hs = p.bs, p.L, p.ulysses, p.ring, p.hs
    hq, hkv, Lq, r, u = p.hc // U, p.hk // U, L // R, rank // U, rank % U
    qh = torch.zeros((U * R, bs, Lq, hq, hs), device="cuda", dtype=torch.bfloat16)
    kh, vh = (torch.zeros((U * R, bs, Lq, hkv, hs), device="cuda", dtype=torch.bfloat16) for _ in range(2))
    for heads, src, dst in ((p.hc, q, qh), (p.hk, k, kh), (p.hk, v, vh)):
        usp.usp_layout_a2a(p, heads, usp.USP_SEQ_TO_HEAD, src, dst, 0, U * R)
    pos = [usp.usp_local_positions(p, s, u)[1] for s in range(R)]
    steps = [(r - i) % R for i in range(R)]
    o, lse = torch.zeros_like(qh[0]), torch.zeros((bs, hq, Lq), device="cuda")
    usp.usp_ring_attn_fwd(qh[rank], [kh[s * U + u] for s in steps], [vh[s * U + u] for s in steps], [pos[s] for s in steps], o, lse, bs,
                          Lq, Lq, hq, hkv, hs, 0.0, p.causal, pos[r], usp.USP_BF16, usp.USP_BF16)
    return o, lse


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_forward_in_place_is_bitwise_the_staged_one(shape):
    L, hc, hk, U, R, hs, causal, zigzag, cut = shape
    N = U * R
    p = usp.problem(1, L, hc, hk, hs, U, R, causal, usp.USP_SPLIT_ZIGZAG if zigzag else usp.USP_SPLIT_CONTIG, usp.USP_BF16)
    gen = torch.Generator(device="cuda").manual_seed(11)
    q = torch.randn((N, 1, L // N, hc, hs), generator=gen, device="cuda", dtype=torch.bfloat16)
    k, v = (torch.randn((N, 1, L // N, hk, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    ws = torch.empty(max(256, usp.usp_attn_fwd_workspace_bytes(p, 1)), dtype=torch.uint8, device="cuda")

    def forward(rank, k, v):
        o, lse = torch.zeros_like(q), torch.zeros((N, 1, hc // U, L // R), device="cuda")
        usp.usp_attn_fwd(p, q, k, v, o, lse, rank, rank + 1, ws)
        head = torch.zeros((N, 1, L // R, hc // U, hs), device="cuda", dtype=torch.bfloat16)
        usp.usp_layout_a2a(p, hc, usp.USP_SEQ_TO_HEAD, o, head, rank, rank + 1)
        return head[rank], lse[rank]

    for rank in sorted({0, N - U, N - 1}):
        o, lse = forward(rank, k, v)
        if shape in ROWS_STAGED:
            staged_o, staged_lse = forward(rank, shifted(k), shifted(v))
            assert torch.equal(o.view(torch.int16), staged_o.view(torch.int16)) and torch.equal(lse, staged_lse)
        else:
            with pytest.raises(usp.UspError) as refused:
                forward(rank, shifted(k), shifted(v))
            assert refused.value.status == 6      # USP_ERR_UNSUPPORTED, as it always was
        dense_o, dense_lse = dense_forward(p, q, k, v, rank)
        if cut.startswith("whole"):
            assert torch.equal(o.view(torch.int16), dense_o.view(torch.int16)) and torch.equal(lse, dense_lse)
        else:   # the pieces' weights are rounded to bf16 against other maxima, and O once more: a few roundings of 2^-9
            assert ((o.double() - dense_o.double()).norm() / dense_o.double().norm()).item() < 2 ** -7
            assert (lse - dense_lse).abs().max().item() < 1e-4


# one writer per element (bf16 from the kernels) / copies; several head splits; ragged tiles; head size 64; batch of two at
# Ulysses degree 1; no mask; more ranks than query tiles
BWD = [(1, 1024, 8, 4, 2, 2, 128, True, True), (1, 3008, 32, 8, 1, 8, 128, True, True), (1, 4 * 550, 16, 8, 4, 1, 64, True, False),
       (2, 1200, 8, 8, 1, 4, 64, False, True), (1, 4096, 32, 32, 2, 4, 128, True, True), (1, 2880, 8, 1, 1, 5, 128, False, False)]


@pytest.mark.parametrize("bs,L,hc,hk,U,R,hs,causal,zigzag", BWD)
def test_backward_of_all_ranks_is_that_of_each_rank(bs, L, hc, hk, U, R, hs, causal, zigzag):
    """All ranks in one call against the sum over one-rank calls (dK, dV: every rank's share, in double), in place and from
    tensors that have to be staged.  Only the order of fp32 sums differs, so two results are at most one rounding to bf16
    apart (2^-8 of a value): 2^-8 on the whole; the sum over ranks adds R values that were rounded on their own."""
    N = U * R
    p = usp.problem(bs, L, hc, hk, hs, U, R, causal, usp.USP_SPLIT_ZIGZAG if zigzag else usp.USP_SPLIT_CONTIG, usp.USP_BF16)
    gen = torch.Generator(device="cuda").manual_seed(5)

    def normal(heads):
        return torch.randn((N, bs, L // N, heads, hs), generator=gen, device="cuda", dtype=torch.bfloat16)

    q, k, v, do = normal(hc), normal(hk), normal(hk), normal(hc)
    o = torch.zeros_like(q)
    lse = torch.zeros((N, bs, hc // U, L // R), device="cuda")
    usp.usp_attn_fwd(p, q, k, v, o, lse, 0, N, torch.empty(max(256, usp.usp_attn_fwd_workspace_bytes(p, N)), dtype=torch.uint8, device="cuda"))

    def backward(begin, end, tensors, workspace_bytes):
        ws = torch.full((workspace_bytes(p, end - begin),), 0xFF, dtype=torch.uint8, device="cuda")
        out = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
        usp.usp_attn_bwd(p, *tensors[:3], tensors[3], lse, tensors[4], *out, begin, end, ws)
        return out

    def apart(x, y):
        return ((x.double() - y.double()).norm() / y.double().norm()).item()

    for need in (usp.usp_attn_bwd_workspace_bytes, usp.usp_attn_bwd_workspace_bytes_with_ds):
        whole = backward(0, N, (q, k, v, o, do), need)
        dq = torch.zeros_like(q)
        dk, dv = (torch.zeros_like(k, dtype=torch.float64) for _ in range(2))
        for rank in range(N):
            one = backward(rank, rank + 1, (q, k, v, o, do), need)
            dq += one[0]      # a rank's rows and heads only: the other elements are zero
            dk += one[1].double()
            dv += one[2].double()
        assert apart(whole[0], dq) < 2 ** -8
        assert apart(whole[1], dk) < 2 ** -8 and apart(whole[2], dv) < 2 ** -8
        if U > 1:
            staged = backward(N - 1, N, (shifted(q), shifted(k), shifted(v), shifted(o), shifted(do)), need)
            for a, b in zip(backward(N - 1, N, (q, k, v, o, do), need), staged):
                assert apart(a, b) < 2 ** -8
