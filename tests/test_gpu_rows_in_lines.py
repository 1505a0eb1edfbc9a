"""Finished rows that leave a workgroup in whole lines, exchanged through LDS: cut forwards (their partial results and the rows
that no cut touches) and the backward's gradients.  Lengths that end inside a wave's 32 rows, outputs that begin at an odd
element, nothing written in front of or behind them, the same bits as outputs of their own."""
import pytest
import torch

import paper_2405_07719_amd as usp
from tests.host_side import HostSide, problem

# L, query and KV heads, head size, Ulysses degree of forwards that are cut, with whole items beside the pieces
CUT = [(4470, 4, 2, 128, 1), (3330, 8, 2, 128, 1), (3100, 16, 8, 64, 1), (5010, 8, 4, 64, 1), (5000, 16, 8, 64, 2)]
# and of short ones, in the launch that splits keys over waves
SHORT = [(L, 4, 2, hs, U) for L, U in ((2590, 1), (4100, 1), (3100, 2), (4100, 2)) for hs in (64, 128)]


def between_guards(t, at):
    """Room for t's shape that begins `at` elements into a buffer of sevens."""
    buf = torch.full((t.numel() + at + 64,), 7.0, dtype=t.dtype, device=t.device)
    return buf, buf[at:at + t.numel()].view(t.shape)


def check(buf, view, at, own):
    assert torch.equal(view, own)
    assert (buf[:at] == 7.0).all() and (buf[at + own.numel():] == 7.0).all()


def test_routes(tmp_path):
    host = HostSide(tmp_path)
    for L, hc, hk, hs, U in CUT + SHORT:
        route = host.forward(problem(1, L, hc, hk, hs, U, 1), 0, 1)
        assert route["kind"] == ("listed" if (L, hc, hk, hs, U) in CUT else "waves"), (L, hs, U, route)
        assert (L, hc, hk, hs, U) in SHORT or (route["whole"] > 0 and route["cut"] > 0), (L, hs, U, route)


@pytest.mark.gpu
@pytest.mark.parametrize("L,hc,hk,hs,U", CUT + SHORT)
def test_forward(L, hc, hk, hs, U):
    gen = torch.Generator(device="cuda").manual_seed(L)
    q = torch.randn((U, 1, L // U, hc, hs), generator=gen, device="cuda", dtype=torch.bfloat16)
    k, v = (torch.randn((U, 1, L // U, hk, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    p = usp.problem(1, L, hc, hk, hs, U, 1, True, usp.USP_SPLIT_ZIGZAG, usp.USP_BF16)
    ws = torch.full((max(256, usp.usp_attn_fwd_workspace_bytes(p, 1)),), 255, dtype=torch.uint8, device="cuda")
    own, lse = torch.zeros_like(q), torch.zeros((U, 1, hc // U, L), device="cuda")
    for rank in range(U):
        usp.usp_attn_fwd(p, q, k, v, own, lse, rank, rank + 1, ws)
    for at in (1, 3, 8):
        buf, o = between_guards(own, at)
        for rank in range(U):
            usp.usp_attn_fwd(p, q, k, v, o, lse, rank, rank + 1, ws)
        check(buf, o, at, own)
    # against double precision: weights and O rounded to bf16, 2^-9 relative each
    qd, kd, vd = (x.double().transpose(0, 1).reshape(L, -1, hs) for x in (q, k, v))
    hidden = torch.ones((L, L), dtype=torch.bool, device="cuda").triu(1)
    got = own.double().transpose(0, 1).reshape(L, hc, hs)
    for h in range(0, hc, 3):
        j = h // (hc // hk)
        ref = (qd[:, h] @ kd[:, j].T * hs ** -0.5).masked_fill(hidden, float("-inf")).softmax(-1) @ vd[:, j]
        assert ((got[:, h] - ref).norm() / ref.norm()).item() < 2 ** -7


@pytest.mark.gpu
@pytest.mark.parametrize("hs", [64, 128])
@pytest.mark.parametrize("L", [40, 1030, 2590])
def test_gradients(L, hs):
    gen = torch.Generator(device="cuda").manual_seed(L)
    q, do = (torch.randn((1, 1, L, 4, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    k, v = (torch.randn((1, 1, L, 2, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    p = usp.problem(1, L, 4, 2, hs, 1, 1, True, usp.USP_SPLIT_ZIGZAG, usp.USP_BF16)
    o, lse = torch.zeros_like(q), torch.zeros((1, 1, 4, L), device="cuda")
    usp.usp_attn_fwd(p, q, k, v, o, lse, 0, 1, torch.empty(max(256, usp.usp_attn_fwd_workspace_bytes(p, 1)), dtype=torch.uint8, device="cuda"))
    for need in (usp.usp_attn_bwd_workspace_bytes, usp.usp_attn_bwd_workspace_bytes_with_ds):
        ws = torch.full((max(256, need(p, 1)),), 255, dtype=torch.uint8, device="cuda")
        own = [torch.zeros_like(x) for x in (q, k, v)]
        usp.usp_attn_bwd(p, q, k, v, o, lse, do, *own, 0, 1, ws)
        for at in (1, 8):
            bufs = [between_guards(x, at) for x in own]
            usp.usp_attn_bwd(p, q, k, v, o, lse, do, *[x for _, x in bufs], 0, 1, ws)
            for (buf, x), y in zip(bufs, own):
                check(buf, x, at, y)
    # fp32 gradients of one block, added to what is there
    delta = torch.zeros((1, 4, L), device="cuda")
    usp.usp_attn_delta(o[0], do[0], delta, 1, L, 4, hs)
    pos = usp.usp_local_positions(p, 0, 0)[1]
    fresh = [torch.zeros_like(x[0], dtype=torch.float32) for x in (q, k, v)]
    usp.usp_ring_attn_bwd(q[0], [k[0]], [v[0]], [pos], do[0], lse[0], delta, fresh[0], [fresh[1]], [fresh[2]], 1, L, L, 4, 2, hs, 0.0, True,
                          pos, False, [False])
    for x, y in zip(fresh, own):
        assert ((x - y[0].float()).norm() / x.norm()).item() < 2 ** -7   # (bf16 results, and other cuts of the sums)
    at = 1
    bufs = [between_guards(x, at) for x in fresh]
    for _, x in bufs:
        x.fill_(0.5)
    (_, dq), (_, dk), (_, dv) = bufs
    usp.usp_ring_attn_bwd(q[0], [k[0]], [v[0]], [pos], do[0], lse[0], delta, dq, [dk], [dv], 1, L, L, 4, 2, hs, 0.0, True, pos, True, [True])
    for (buf, x), y in zip(bufs, fresh):
        # one rounding to fp32 of a sum of 0.5 and a gradient, more where split heads meet by atomic additions
        assert torch.allclose(x, y + 0.5, rtol=0, atol=1e-5 * max(1.0, y.abs().max().item()))
        assert (buf[:at] == 7.0).all() and (buf[at + y.numel():] == 7.0).all()
