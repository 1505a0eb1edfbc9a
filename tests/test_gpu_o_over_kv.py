"""The forward with O (or LSE) in the memory of K, of V or of Q: what the same call gives with results of their own.  Every
rank of the range reads all of K and V, so nothing of it may be written before the last of them has read."""
import pytest
import torch

import paper_2405_07719_amd as usp

pytestmark = pytest.mark.gpu

BF16, FP32 = usp.USP_BF16, usp.USP_FP32
# bs, L, heads, U, R, hs, causal, dtype, one rank or all
SHAPES = [
    (1, 16384, 16, 2, 1, 128, True, BF16, False),    # whole items, V re-tiled or as rows
    (1, 12288, 8, 2, 2, 128, True, BF16, False),     # a ring of two
    (1, 10240, 32, 8, 1, 128, True, BF16, True),     # heaviest tiles cut
    (1, 4608, 8, 2, 1, 64, False, BF16, True),       # every tile cut, or all ranks in one launch
    (2, 1024, 8, 2, 2, 128, True, BF16, False),      # short, a batch of two
    (1, 1024, 8, 4, 1, 64, True, BF16, False),       # short, a batch of one
    (1, 40 * 32, 4, 2, 20, 64, True, BF16, False),   # more ring blocks than one launch takes
    (1, 1088, 8, 2, 2, 64, True, FP32, False),
    (2, 512, 4, 4, 1, 128, False, FP32, False),
    (1, 704, 4, 1, 1, 64, True, FP32, True),         # Ulysses degree 1: one fp32 rank
    (2, 1024, 4, 1, 4, 128, True, FP32, True),
]


# Ulysses degree 1: K and V are read where they lie, but for O of one fp32 rank; that rank's Q is copied, too
CASES = [(*s, over) for s in SHAPES for over in ("k", "v", "q", "lse over k", "half of q")
         if (over != "half of q" or s[7] == FP32 and s[8]) and (over != "lse over k" or s[3] > 1)]


@pytest.mark.parametrize("bs,L,heads,U,R,hs,causal,dtype,one,over", CASES)
def test_results_over_inputs(bs, L, heads, U, R, hs, causal, dtype, one, over):
    N, torch_dtype = U * R, torch.float32 if dtype == FP32 else torch.bfloat16
    split = usp.USP_SPLIT_ZIGZAG if L % (2 * N) == 0 else usp.USP_SPLIT_CONTIG
    p = usp.problem(bs, L, heads, heads, hs, U, R, causal, split, dtype)
    begin, end = (N - 1, N) if one else (0, N)
    gen = torch.Generator(device="cuda").manual_seed(L)
    shape = (N, bs, L // N, heads, hs)
    ws = torch.empty(max(256, usp.usp_attn_fwd_workspace_bytes(p, end - begin)), dtype=torch.uint8, device="cuda")

    def call(place):
        gen.manual_seed(L)
        n = N * bs * (L // N) * heads * hs
        long = torch.zeros(2 * n, device="cuda", dtype=torch_dtype)   # Q, and room behind it
        q = long[:n].view(shape).copy_(torch.randn(shape, generator=gen, device="cuda", dtype=torch_dtype))
        k, v = (torch.randn(shape, generator=gen, device="cuda", dtype=torch_dtype) for _ in range(2))
        o = {"k": k, "v": v, "q": q, "half of q": long[n // 2:n // 2 + n].view(shape)}.get(place)
        o = torch.zeros_like(q) if o is None else o
        lse_shape = (N, bs, heads // U, L // R)
        lse = torch.zeros(lse_shape, device="cuda")
        if place == "lse over k":
            lse = k.view(-1).view(torch.float32)[:lse.numel()].view(lse_shape)
        usp.usp_attn_fwd(p, q, k, v, o, lse, begin, end, ws)
        return o, lse

    ref_o, ref_lse = call(None)
    o, lse = call(over)
    r0, r1 = begin // U * U, ((end - 1) // U + 1) * U       # the ring rows written to
    head = slice((N - 1) % U * (heads // U), heads) if one else slice(0, heads)
    x, y = o[r0:r1, :, :, head].double(), ref_o[r0:r1, :, :, head].double()
    # P and the partial results are rounded to bf16 at other places where the route differs (a few roundings of 2^-9); fp32
    # sums of up to 2^11 terms in another order: 2^-24 sqrt(2^11) is 3e-6
    assert ((x - y).norm() / y.norm()).item() < (1e-5 if dtype == FP32 else 2 ** -7)
    assert (lse[begin:end].double() - ref_lse[begin:end].double()).abs().max().item() < (1e-5 if dtype == FP32 else 1e-4)
