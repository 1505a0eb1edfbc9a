"""Ring ranks of the zigzag split whose two runs of rows do not end on a whole tile: no 256-row tile of the attention
kernels holds rows (or keys) of both runs.  One rank, forward and backward, against double precision."""
import pytest
import torch

import paper_2405_07719_amd as usp

pytestmark = pytest.mark.gpu

# rows of a run: shorter than a wave, one short of / one past a tile, several tiles and a remainder, a whole tile
CHUNKS = [(20, 2), (255, 2), (257, 3), (300, 4), (513, 2), (256, 2), (1000, 2)]


@pytest.mark.parametrize("hs", [64, 128])
@pytest.mark.parametrize("c,R", CHUNKS)
def test_rows_of_two_runs(c, R, hs):
    hq, hkv, L, Lq = 4, 2, 2 * R * c, 2 * c
    gen = torch.Generator(device="cuda").manual_seed(c)
    q, do = (torch.randn((1, Lq, hq, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    k, v = ([torch.randn((1, Lq, hkv, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(R)] for _ in range(2))
    p = usp.problem(1, L, hq, hkv, hs, 1, R, True, usp.USP_SPLIT_ZIGZAG, usp.USP_BF16)
    pos = [usp.usp_local_positions(p, s, 0)[1] for s in range(R)]
    r = R - 1
    o = torch.zeros((1, Lq, hq, hs), device="cuda", dtype=torch.bfloat16)
    lse = torch.zeros((1, hq, Lq), device="cuda")
    usp.usp_ring_attn_fwd(q, k, v, pos, o, lse, 1, Lq, Lq, hq, hkv, hs, 0.0, True, pos[r], usp.USP_BF16, usp.USP_BF16)

    def runs(d):
        return torch.cat([torch.arange(d.start0, d.start0 + d.len0), torch.arange(d.start1, d.start1 + d.len1)]).cuda()

    hidden = torch.cat([runs(d) for d in pos])[None, :] > runs(pos[r])[:, None]
    kd, vd = (torch.cat([x[0] for x in t]).double().repeat_interleave(hq // hkv, 1) for t in (k, v))
    qd, dod = q[0].double(), do[0].double()
    ref = {n: torch.zeros_like(x) for n, x in (("o", qd), ("dq", qd), ("dk", kd), ("dv", kd))}
    for h in range(hq):
        w = (qd[:, h] @ kd[:, h].T * hs ** -0.5).masked_fill(hidden, float("-inf")).softmax(-1)
        ref["o"][:, h] = w @ vd[:, h]
        ds = w * (dod[:, h] @ vd[:, h].T - (dod[:, h] * ref["o"][:, h]).sum(-1, keepdim=True))
        ref["dq"][:, h], ref["dk"][:, h], ref["dv"][:, h] = ds @ kd[:, h] * hs ** -0.5, ds.T @ qd[:, h] * hs ** -0.5, w.T @ dod[:, h]

    def far(x, y):
        return ((x.double() - y).norm() / y.norm()).item()

    # weights, dS and O rounded to bf16 (2^-9 relative each, a few of them on the way to a gradient): below 2^-7
    assert far(o[0], ref["o"]) < 2 ** -7
    delta = torch.zeros((1, hq, Lq), device="cuda")
    usp.usp_attn_delta(o, do, delta, 1, Lq, hq, hs)
    dq = torch.full((1, Lq, hq, hs), float("nan"), device="cuda")
    dk, dv = ([torch.full((1, Lq, hkv, hs), float("nan"), device="cuda") for _ in range(R)] for _ in range(2))
    usp.usp_ring_attn_bwd(q, k, v, pos, do, lse, delta, dq, dk, dv, 1, Lq, Lq, hq, hkv, hs, 0.0, True, pos[r], False, [False] * R)
    assert far(dq[0], ref["dq"]) < 2 ** -7
    for got, n in ((dk, "dk"), (dv, "dv")):
        assert far(torch.cat([x[0] for x in got]), ref[n].view(R * Lq, hkv, hq // hkv, hs).sum(2)) < 2 ** -7
