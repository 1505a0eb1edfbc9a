"""Ring ranks of the zigzag split whose two runs of rows do not end on a whole tile: where tl.cut_apart() says so, no
256-row tile of the forward holds rows of both runs, nor one of the backward's query tiles (one rank's rows), nor one of its
key tiles where a call has the one block; the last ring rank's runs adjoin, so that a call with all blocks has their keys in a
row.  Every rank, forward and backward, against double precision."""
import pytest
import torch

import paper_2405_07719_amd as usp
from tests import usp_testlib as tl

pytestmark = pytest.mark.gpu

# rows of a run: shorter than a wave, one short of / one past a tile, several tiles and a remainder, a whole tile; cut apart
# without a tile more (the first row) and with one more (1030: a second tile of six rows)
APART = [(255, 2), (255, 4), (1000, 2), (1100, 2), (1030, 3)]
IN_A_ROW = [(20, 2), (257, 3), (300, 4), (513, 2), (256, 2)]


@pytest.mark.parametrize("hs", [64, 128])
@pytest.mark.parametrize("c,R,r", [(c, R, r) for c, R in APART + IN_A_ROW for r in range(R)])
def test_rows_of_two_runs(c, R, r, hs):
    hq, hkv, L, Lq = 4, 2, 2 * R * c, 2 * c
    assert tl.cut_apart(c, R, r) == ((c, R) in APART and r < R - 1)
    gen = torch.Generator(device="cuda").manual_seed(c)
    q, do = (torch.randn((1, Lq, hq, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    k, v = ([torch.randn((1, Lq, hkv, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(R)] for _ in range(2))
    p = usp.problem(1, L, hq, hkv, hs, 1, R, True, usp.USP_SPLIT_ZIGZAG, usp.USP_BF16)
    pos = [usp.usp_local_positions(p, s, 0)[1] for s in range(R)]
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
    sums = {n: ref[n].view(R * Lq, hkv, hq // hkv, hs).sum(2) for n in ("dk", "dv")}
    for got, n in ((dk, "dk"), (dv, "dv")):
        assert far(torch.cat([x[0] for x in got]), sums[n]) < 2 ** -7
    # block by block: key tiles, too, end with a run
    dq.zero_()
    for x in dk + dv:
        x.zero_()
    for s in range(R):
        usp.usp_block_attn_bwd(q, k[s], v[s], do, lse, delta, dq, dk[s], dv[s], 1, Lq, Lq, hq, hkv, hs, 0.0, True, pos[r], pos[s], True)
    assert far(dq[0], ref["dq"]) < 2 ** -7
    for got, n in ((dk, "dk"), (dv, "dv")):
        assert far(torch.cat([x[0] for x in got]), sums[n]) < 2 ** -7


@pytest.mark.parametrize("bs,L,hc,hk,hs", [
    (1, 17600, 16, 4, 128),      # the heaviest tiles cut (the last 14 of 18 of the second run), V as rows
    (1, 37280, 16, 4, 128),      # the same, V in transposed tiles
    (1, 4400, 128, 16, 128),     # whole items, K and V in place
    (2, 4400, 64, 16, 128),      # whole items, K staged, V in transposed tiles, a batch of two
    (1, 4400, 128, 16, 64),
    (1, 4400, 16, 4, 128),       # every tile cut
])
def test_forward_on_the_shards(bs, L, hc, hk, hs):
    """usp_attn_fwd, first rank of each ring row of Ulysses 2 x ring 2: rows around the ends of runs and tiles, and others,
    against double precision; both rows of ranks, so that every element of the shards has been written."""
    U, R, c = 2, 2, L // 4
    assert tl.cut_apart(c, R, 0) and not tl.cut_apart(c, R, 1)
    p = usp.problem(bs, L, hc, hk, hs, U, R, True, usp.USP_SPLIT_ZIGZAG, usp.USP_BF16)
    gen = torch.Generator(device="cuda").manual_seed(L)
    q, k, v = (torch.randn((U * R, bs, L // 4, h, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hc, hk, hk))
    o = torch.full_like(q, float("nan"))
    lse = torch.full((U * R, bs, hc // U, L // R), float("nan"), device="cuda")
    ws = torch.empty(max(256, usp.usp_attn_fwd_workspace_bytes(p, 1)), dtype=torch.uint8, device="cuda")
    for rank in range(U * R):
        usp.usp_attn_fwd(p, q, k, v, o, lse, rank, rank + 1, ws)
    assert torch.isfinite(o).all() and torch.isfinite(lse).all()

    def block(t, r, b):      # [L/R, heads, hs]: the rows of ring row r
        return torch.cat([t[r * U + u, b] for u in range(U)])

    b, Lq, g = bs - 1, L // R, hc // hk
    pos = [torch.cat([torch.arange(r * c, (r + 1) * c), torch.arange((3 - r) * c, (4 - r) * c)]).cuda() for r in range(R)]
    kpos = torch.cat(pos)
    for r in range(R):
        rows = {i + d for i in (0, 256, c // 256 * 256, c, c + 256, c + c // 256 * 256, Lq) for d in (-2, -1, 0, 1)} | set(range(5, Lq, 97))
        rows = torch.tensor(sorted(i for i in rows if 0 <= i < Lq), device="cuda")
        hidden = kpos[None, :] > pos[r][rows][:, None]
        for h in (0, hc - 1):
            qd, od = (block(t, r, b)[rows, h].double() for t in (q, o))
            kd, vd = (torch.cat([block(t, s, b)[:, h // g] for s in range(R)]).double() for t in (k, v))
            scores = (qd @ kd.T * hs ** -0.5).masked_fill(hidden, float("-inf"))
            want = scores.softmax(-1) @ vd
            # a row's O against its own size: weights and O rounded to bf16
            assert ((od - want).norm(dim=-1) / want.norm(dim=-1)).max().item() < 2 ** -6
            u = h // (hc // U)
            assert (lse[r * U + u, b, h % (hc // U)][rows].double() - scores.logsumexp(-1)).abs().max().item() < 1e-4
