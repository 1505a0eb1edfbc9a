"""The forward at head size 64, whose second product runs a tile behind in blocks of 2048 keys and more, and which forms row
maxima there only where the weights leave their bound: one to seven key tiles and ragged ones, scores that grow and fall by
thousands of powers of two from tile to tile, rows that see nothing, several blocks, V in transposed tiles, cut forwards, the running
state; the routes on the CPU.  Against double precision."""
import pytest
import torch

import paper_2405_07719_amd as usp
from tests.host_side import HostSide, problem

HS = 64


def reference(q, k, v, qpos, kpos, causal):
    s = torch.einsum("ihd,jhd->hij", q.double(), k.double().repeat_interleave(q.shape[1] // k.shape[1], 1)) * HS ** -0.5
    if causal:
        s = s.masked_fill((kpos[None, :] > qpos[:, None])[None], float("-inf"))
    lse = s.logsumexp(-1)
    w = torch.exp(s - torch.where(lse.isinf(), torch.zeros_like(lse), lse)[..., None])
    return torch.einsum("hij,jhd->ihd", w, v.double().repeat_interleave(q.shape[1] // v.shape[1], 1)), lse


def compare(o, lse, ref_o, ref_lse):
    # weights and O rounded to bf16, 2^-9 relative each
    assert ((o.double() - ref_o).norm() / ref_o.norm()).item() < 2 ** -7
    seen = ref_lse.isfinite()
    assert torch.equal(lse.isfinite(), seen)
    # scores are sums of 64 fp32 products: a few roundings of the largest
    assert ((lse.double() - ref_lse)[seen].abs() <= 1e-6 * ref_lse[seen].abs().max().clamp(min=4.0)).all()


# factors of the scores of one key tile after the other
STEPS = {"even": [1.0] * 7, "growing": [0.01, 0.3, 1, 10, 100, 300, 1000], "falling": [1000, 100, 10, 1, 0.1, 0.01, 0.0],
         "up and down": [0.0, 50, 0.1, 500, 0.0, 5000, 1.0]}


def transposed(v):
    """A block's V [1][keys][heads][64] in transposed tiles."""
    _, Lk, hkv, _ = v.shape
    t = torch.full((1, hkv, (Lk + 63) // 64, HS, 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    usp.usp_layout_a2a(usp.problem(1, Lk, hkv, hkv, HS, 1, 1, False, usp.USP_SPLIT_CONTIG, usp.USP_BF16), hkv, usp.USP_SEQ_TO_HEAD_VT, v, t, 0, 1)
    return t


def rings(k, v, q, qd, causal, how):
    """One block, and two; the second lies behind the first."""
    Lk, Lq, hq, hkv = k.shape[1], q.shape[0], q.shape[1], k.shape[2]
    k = (k.float() * torch.tensor(STEPS[how], device="cuda").repeat_interleave(64).repeat(-(-Lk // 448))[:Lk, None, None]).bfloat16()
    first, second = usp.usp_posdesc(5, Lk, 0, 0), usp.usp_posdesc(Lk + 5, Lk, 0, 0)
    qpos, kpos = torch.arange(qd.start0, qd.start0 + Lq).cuda(), torch.arange(2 * Lk).cuda() + 5
    for n in (1, 2):
        o, lse = torch.full((1, Lq, hq, HS), float("nan"), device="cuda").bfloat16(), torch.full((1, hq, Lq), float("nan"), device="cuda")
        ks, vs = [k[j].contiguous()[None] for j in range(n)], [v[j].contiguous()[None] for j in range(n)]
        usp.usp_ring_attn_fwd(q[None], ks, vs, [first, second][:n], o, lse, 1, Lq, Lk, hq, hkv, HS, 0.0, causal, qd, usp.USP_BF16, usp.USP_BF16)
        compare(o[0], lse[0], *reference(q, k[:n].flatten(0, 1), v[:n].flatten(0, 1), qpos, kpos[:n * Lk], causal))
        # V in transposed tiles: the same products in the same order
        o1, lse1 = torch.full_like(o, float("nan")), torch.full_like(lse, float("nan"))
        usp.usp_ring_attn_fwd_vt(q[None], ks, [transposed(x) for x in vs], [first, second][:n], o1, lse1, 1, Lq, Lk, hq, hkv, HS, 0.0, causal, qd)
        assert torch.equal(o1.view(torch.int16), o.view(torch.int16)) and torch.equal(lse1.view(torch.int32), lse.view(torch.int32))


def draw(seed, Lq, Lk):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q = torch.randn((Lq, 4, HS), generator=gen, device="cuda").bfloat16()
    return q, *(torch.randn((2, Lk, 2, HS), generator=gen, device="cuda").bfloat16() for _ in range(2))


# short blocks (the loop without the tile behind) and long ones, whole and ragged; the rows begin ahead of the first key
@pytest.mark.gpu
@pytest.mark.parametrize("how", STEPS)
@pytest.mark.parametrize("Lk", [1, 65, 192, 320, 447, 2048, 2049, 2300])
@pytest.mark.parametrize("causal", [False, True])
def test_one_block_and_two(Lk, how, causal):
    q, k, v = draw(Lk, 300, Lk)
    rings(k, v, q, usp.usp_posdesc(0, 300, 0, 0), causal, how)


# long blocks of which the last row sees one to seven tiles, up to a key past a tile
@pytest.mark.gpu
@pytest.mark.parametrize("how", STEPS)
@pytest.mark.parametrize("seen", [1, 63, 64, 65, 128, 130, 192, 200, 256, 300, 320, 447])
def test_few_tiles_of_a_long_block(seen, how):
    Lq = min(seen + 5, 290)
    q, k, v = draw(seen, Lq, 2100)
    rings(k, v, q, usp.usp_posdesc(seen + 5 - Lq, Lq, 0, 0), True, how)


# Maxima that move twice within a few tiles are watched for 32 tiles after the last move: moves from one tile to the next, at 12
# tiles' distance and at 13, the last one in the last tile, calm in between and at the end; a mask, a ragged tail, a second block.
MOVES = {"once": [0], "close, then calm": [0, 3, 4, 5], "twelve and thirteen apart": [0, 12, 25, 37, 50], "every second tile": range(0, 70, 2),
         "calm, then close": [0, 45, 46, 47], "to the last tile": [0, 2, 34, 66, 69], "watched to the end": [0, 60, 68]}


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("moves", MOVES)
@pytest.mark.parametrize("Lk", [70 * 64, 69 * 64 + 5])
def test_maxima_that_move_often(Lk, moves, causal):
    q, k, v = draw(Lk, 290, Lk)
    f, height = [], 1.0
    for tile in range(70):
        if tile in MOVES[moves]:
            height *= 1.6 if len(MOVES[moves]) > 6 else 4.0
        f.append(height if tile in MOVES[moves] else 0.3 * height)
    k = (k.float() * torch.tensor(f, device="cuda").repeat_interleave(64)[:Lk, None, None]).bfloat16()
    qd, first, second = usp.usp_posdesc(Lk - 150, 290, 0, 0), usp.usp_posdesc(0, Lk, 0, 0), usp.usp_posdesc(Lk, Lk, 0, 0)
    qpos, kpos = torch.arange(Lk - 150, Lk + 140).cuda(), torch.arange(2 * Lk).cuda()
    o, lse = torch.full((1, 290, 4, HS), float("nan"), device="cuda").bfloat16(), torch.full((1, 4, 290), float("nan"), device="cuda")
    usp.usp_ring_attn_fwd(q[None], [k[:1], k[1:]], [v[:1], v[1:]], [first, second], o, lse, 1, 290, Lk, 4, 2, HS, 0.0, causal, qd, usp.USP_BF16,
                          usp.USP_BF16)
    compare(o[0], lse[0], *reference(q, k.flatten(0, 1), v.flatten(0, 1), qpos, kpos, causal))


def factors(how, n):
    """Of the scores of n keys."""
    return torch.tensor(STEPS[how], device="cuda").repeat_interleave(64).repeat(-(-n // 448))[:n, None, None]


# Batch, L, query and KV heads, Ulysses and ring degree, mask; the launch, V in transposed tiles.  Long enough for the tile behind.
WHOLE = [((1, 8850, 4, 4, 1, 1, True), "listed", 0), ((1, 9004, 8, 2, 1, 2, True), "listed", 0), ((2, 9004, 8, 8, 2, 1, False), "listed", 1),
         ((2, 6200, 8, 2, 2, 1, False), "whole", 1), ((1, 5204, 16, 16, 1, 2, False), "whole", 0)]


def test_routes(tmp_path):
    host = HostSide(tmp_path)
    for (bs, L, hc, hk, U, R, causal), kind, v_transposed in WHOLE:
        route = host.forward(problem(bs, L, hc, hk, HS, U, R, causal), 0, 1)
        assert (route["kind"], route["v_transposed"]) == (kind, v_transposed), (L, route)
        assert L // R >= 2048 and (kind == "whole" or L // route["parts"] >= 1250), (L, route)
    for h, n in STATES:
        assert not host.lib.block_goes_to_waves(1, host.long(n), host.long(n), h, HS, 1, usp.USP_BF16)


@pytest.mark.gpu
@pytest.mark.parametrize("how", STEPS)
@pytest.mark.parametrize("shape", [x for x, _, _ in WHOLE], ids=str)
def test_whole_forward(shape, how):
    bs, L, hc, hk, U, R, causal = shape
    gen = torch.Generator(device="cuda").manual_seed(L)
    p = usp.problem(bs, L, hc, hk, HS, U, R, causal, usp.USP_SPLIT_ZIGZAG, usp.USP_BF16)
    N, h = U * R, hc // U
    q, k, v = (torch.randn((N, bs, L // N, n, HS), generator=gen, device="cuda").bfloat16() for n in (hc, hk, hk))
    pos = [usp.usp_local_positions(p, r, 0)[1] for r in range(R)]
    at = [torch.cat([torch.arange(d.start0, d.start0 + d.len0), torch.arange(d.start1, d.start1 + d.len1)]).cuda() for d in pos]
    # (rows of a ring rank: its shards one behind the other; factors by the key's place in them, block after block)
    k = (k.view(R, U, bs, L // N, hk, HS).transpose(1, 2).reshape(R, bs, L // R, hk, HS) * factors(how, L // R)).bfloat16()
    k = k.view(R, bs, U, L // N, hk, HS).transpose(1, 2).reshape(N, bs, L // N, hk, HS).contiguous()
    o, lse = torch.full_like(q, float("nan")), torch.full((N, bs, h, L // R), float("nan"), device="cuda")
    ws = torch.full((max(256, usp.usp_attn_fwd_workspace_bytes(p, 1)),), 255, dtype=torch.uint8, device="cuda")
    for rank in range(N):
        usp.usp_attn_fwd(p, q, k, v, o, lse, rank, rank + 1, ws)
    rows = lambda t, r, b: t.view(R, U, bs, L // N, -1, HS)[r, :, b].flatten(0, 1)
    b, group = bs - 1, hc // hk
    for r in range(R):
        kr, vr = (torch.cat([rows(t, s, b) for s in range(R)]) for t in (k, v))
        for head in (0, hc - 1):
            one = slice(head, head + 1), slice(head // group, head // group + 1)
            compare(rows(o, r, b)[:, one[0]], lse[r * U + head // h, b, head % h][None],
                    *reference(rows(q, r, b)[:, one[0]], kr[:, one[1]], vr[:, one[1]], at[r], torch.cat(at), causal))


# heads, rows and keys of a ring rank: steps that are too much work for one workgroup's waves
STATES = [(32, 2200), (32, 2050)]


@pytest.mark.gpu
@pytest.mark.parametrize("order", [(0, 1), (1, 0)], ids=["own block first", "own block last"])
@pytest.mark.parametrize("how", STEPS)
@pytest.mark.parametrize("h,n", STATES)
def test_running_state(h, n, how, order):
    R, hk = 2, 4
    gen = torch.Generator(device="cuda").manual_seed(7)
    p = usp.problem(1, R * n, h, hk, HS, 1, R, True, usp.USP_SPLIT_ZIGZAG, usp.USP_BF16)
    q = torch.randn((1, n, h, HS), generator=gen, device="cuda").bfloat16()
    k, v = (torch.randn((R, 1, n, hk, HS), generator=gen, device="cuda") for _ in range(2))
    k, v = (k * factors(how, n)).bfloat16(), v.bfloat16()
    pos = [usp.usp_local_positions(p, r, 0)[1] for r in range(R)]
    at = [torch.cat([torch.arange(d.start0, d.start0 + d.len0), torch.arange(d.start1, d.start1 + d.len1)]).cuda() for d in pos]
    for r in range(R):
        state = torch.zeros(usp.usp_block_attn_fwd_state_bytes(1, n, h, HS), dtype=torch.uint8, device="cuda")
        o, lse = torch.full_like(q, float("nan")), torch.full((1, h, n), float("nan"), device="cuda")
        for i, step in enumerate(order):
            s = (r - step) % R
            usp.usp_block_attn_fwd_state(q, k[s], v[s], state, o, lse, 1, n, n, h, hk, HS, 0.0, True, pos[r], pos[s], i == 0, i == R - 1,
                                         usp.USP_BF16)
        for head in (0, 9, 31):
            group = slice(head // 8, head // 8 + 1)
            compare(o[0, :, head:head + 1], lse[0, head:head + 1],
                    *reference(q[0, :, head:head + 1], k[:, 0, :, group].flatten(0, 1), v[:, 0, :, group].flatten(0, 1), at[r], torch.cat(at), True))
