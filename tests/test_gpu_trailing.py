"""The forward at head size 64, whose second product runs a tile behind in blocks of 2048 keys and more, and which forms row
maxima there only where the weights leave their bound: one to seven key tiles and ragged ones, scores that grow and fall by
thousands of powers of two from tile to tile, rows that see nothing, several blocks, the running state.  Against double precision."""
import pytest
import torch

import paper_2405_07719_amd as usp

pytestmark = pytest.mark.gpu
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


def draw(seed, Lq, Lk):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q = torch.randn((Lq, 4, HS), generator=gen, device="cuda").bfloat16()
    return q, *(torch.randn((2, Lk, 2, HS), generator=gen, device="cuda").bfloat16() for _ in range(2))


# short blocks (the loop without the tile behind) and long ones, whole and ragged; the rows begin ahead of the first key
@pytest.mark.parametrize("how", STEPS)
@pytest.mark.parametrize("Lk", [1, 65, 192, 320, 447, 2048, 2049, 2300])
@pytest.mark.parametrize("causal", [False, True])
def test_one_block_and_two(Lk, how, causal):
    q, k, v = draw(Lk, 300, Lk)
    rings(k, v, q, usp.usp_posdesc(0, 300, 0, 0), causal, how)


# long blocks of which the last row sees one to seven tiles, up to a key past a tile
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


@pytest.mark.parametrize("how", STEPS)
@pytest.mark.parametrize("L", [4400, 2200])
def test_running_state_and_whole_forward(L, how):
    R, h = 2, 4
    gen = torch.Generator(device="cuda").manual_seed(7)
    p = usp.problem(1, L, h, h, HS, 1, R, True, usp.USP_SPLIT_ZIGZAG, usp.USP_BF16)
    q, k, v = (torch.randn((R, 1, L // R, h, HS), generator=gen, device="cuda") for _ in range(3))
    f = torch.tensor(STEPS[how], device="cuda").repeat_interleave(64).repeat(-(-L // R // 448))[:L // R]
    q, k, v = q.bfloat16(), (k * f[None, None, :, None, None]).bfloat16(), v.bfloat16()
    pos = [usp.usp_local_positions(p, r, 0)[1] for r in range(R)]
    at = [torch.cat([torch.arange(d.start0, d.start0 + d.len0), torch.arange(d.start1, d.start1 + d.len1)]).cuda() for d in pos]
    o, lse = torch.zeros_like(q), torch.zeros((R, 1, h, L // R), device="cuda")
    usp.usp_attn_fwd(p, q, k, v, o, lse, 0, R, torch.empty(max(256, usp.usp_attn_fwd_workspace_bytes(p, R)), dtype=torch.uint8, device="cuda"))
    for r in range(R):
        ref = reference(q[r, 0], k[:, 0].flatten(0, 1), v[:, 0].flatten(0, 1), at[r], torch.cat(at), True)
        compare(o[r, 0], lse[r, 0], *ref)
        state = torch.zeros(usp.usp_block_attn_fwd_state_bytes(1, L // R, h, HS), dtype=torch.uint8, device="cuda")
        o1, lse1 = torch.zeros_like(o[r]), torch.zeros_like(lse[r])
        for i in range(R):
            s = (r - i) % R
            usp.usp_block_attn_fwd_state(q[r], k[s], v[s], state, o1, lse1, 1, L // R, L // R, h, h, HS, 0.0, True, pos[r], pos[s], i == 0,
                                         i == R - 1, usp.USP_BF16)
        compare(o1[0], lse1[0], *ref)
