"""GPU parity of the forward that splits the keys of 32 rows over the waves of a workgroup: every rank of a problem in one
launch on the sequence-layout shards (short bf16 sequences, fp32 of every size), and one ring step on dense tensors.  The
sizes are the edges of its tiles: rows and keys around 32, tiles that cross from one shard into the next (bs > 1), shards
shorter than a tile, fewer visible tiles than waves, more ring blocks than a launch of the other kernel takes."""
import numpy as np
import pytest
import torch

from oracle import usp_oracle as orc
from tests import usp_testlib as tl
from tests.test_gpu_attn_fwd import BLOCK_CASES, _check_against_reference, _desc, _run_block, _run_usp_fwd  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def usp():
    import paper_2405_07719_amd as pkg
    pkg.load()
    return pkg


@pytest.mark.parametrize("dtype", [tl.BF16, tl.FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("bs,L,hc,hk,hs,U,R,causal,zigzag", [
    (1, 2, 2, 1, 64, 1, 1, True, True),             # two rows in all
    (1, 31, 2, 2, 128, 1, 1, False, False),         # less than a tile
    (2, 66, 2, 1, 64, 1, 1, True, False),           # two tiles and two rows
    (3, 40, 4, 2, 128, 2, 2, True, True),           # shards of 10 rows, blocks of 20: tiles span three shards
    (2, 264, 4, 4, 64, 2, 2, True, True),           # shards of 66 rows: tiles straddle one boundary
    (2, 296, 8, 2, 128, 2, 1, False, False),        # shards of 148 rows, group of four heads
    (1, 1056, 4, 2, 128, 1, 4, True, True),         # runs of 132 positions: a tile holds keys of both runs
    (1, 640, 4, 1, 64, 1, 20, True, True),          # 20 ring blocks of 32 keys
    (1, 1536, 8, 8, 128, 4, 2, True, False),        # contiguous blocks: rank 0 sees nothing of block 1
])
def test_all_ranks_match_the_oracle(usp, dtype, bs, L, hc, hk, hs, U, R, causal, zigzag):
    prob = tl.Problem(900 + L, bs, L, hc, hk, hs, U, R, causal, zigzag, dtype)
    o, lse = _run_usp_fwd(usp, prob)
    ref_o, tol = _check_against_reference(prob, o, lse)
    for rank in range(prob.N):
        assert tl.max_abs(o[rank], ref_o[rank]) <= tol, rank


@pytest.mark.parametrize("dtype", [tl.BF16, tl.FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("bs,L,hc,hk,hs,U,R,causal,zigzag", [
    (2, 330, 4, 2, 64, 1, 5, True, True),           # shards of 66 rows: the second run begins inside a shard's second tile
    (2, 1056, 4, 4, 128, 4, 1, True, True),         # shards of 264: nine tiles each, the last of eight rows
    (3, 1188, 2, 2, 128, 2, 2, False, False),       # shards of 297 without a mask: every ragged tile is masked
    (2, 2112, 4, 2, 64, 2, 3, True, False),         # more tiles than waves in every block, shards of 352 = 11 tiles
    (1, 1036, 4, 2, 64, 2, 1, True, True),          # one run of rows: a batch of one, the last tile of twelve rows
])
def test_tiles_end_with_their_shard(usp, dtype, bs, L, hc, hk, hs, U, R, causal, zigzag):
    """Key tiles at the ends of shards: numbered shard by shard, or crossing once (head size 128, 32 rows per workgroup)."""
    prob = tl.Problem(970 + L, bs, L, hc, hk, hs, U, R, causal, zigzag, dtype)
    o, lse = _run_usp_fwd(usp, prob)
    ref_o, tol = _check_against_reference(prob, o, lse)
    for rank in range(prob.N):
        assert tl.max_abs(o[rank], ref_o[rank]) <= tol, rank


# shards of few rows, whose tiles cross: how often at most (tests/test_wave_split_host.py asks the library's rule)
CROSSING = [
    (2, 96, 4, 4, 128, 4, 4, True, True, 2),        # shards of 6 rows: a tile spans six shards; runs of 12 positions
    (3, 80, 8, 8, 64, 8, 1, False, False, 2),       # of 10 without a mask, a ragged last tile
    (2, 320, 8, 8, 128, 8, 4, False, True, 2),      # of 10, in fp32 with 32 rows per workgroup
    (2, 320, 8, 8, 64, 8, 4, False, True, 2),
    (2, 272, 8, 8, 128, 8, 1, True, True, 1),       # of 34: crossings move through the tile, two rows a shard
    (2, 1088, 8, 8, 64, 8, 4, True, True, 1),       # of 34, more tiles than waves, runs that end inside a tile
    (4, 1088, 8, 8, 128, 8, 4, False, False, 1),
    (2, 1280, 4, 4, 64, 4, 8, True, False, 1),      # of 40: tiles that begin where a shard does
]


@pytest.mark.parametrize("dtype", [tl.BF16, tl.FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("bs,L,hc,hk,hs,U,R,causal,zigzag,cross", CROSSING)
def test_tiles_cross_from_one_shard_into_the_next(usp, dtype, bs, L, hc, hk, hs, U, R, causal, zigzag, cross):
    prob = tl.Problem(930 + L + hs, bs, L, hc, hk, hs, U, R, causal, zigzag, dtype)
    o, lse = _run_usp_fwd(usp, prob)
    ref_o, tol = _check_against_reference(prob, o, lse)
    for rank in range(prob.N):
        assert tl.max_abs(o[rank], ref_o[rank]) <= tol, rank


@pytest.mark.parametrize("hs", [64, 128])
@pytest.mark.parametrize("bs,L,hc,hk,U,R,causal,zigzag", [
    (1, 6, 2, 1, 1, 1, True, True),                 # fewer rows than a workgroup's 16
    (1, 2048, 4, 4, 1, 1, True, True),              # 256 workgroups of 32 rows: the last size with 16 under a mask
    (1, 2080, 4, 4, 1, 1, True, True),              # ... and the first with 32
    (1, 1024, 4, 2, 1, 1, False, True),             # 128: the last with 16 without a mask
    (1, 1048, 4, 2, 1, 1, False, True),             # ... and the first with 32 (ragged: 24 rows in the last)
    (2, 204, 4, 2, 2, 1, True, False),              # shards of 102 rows, row tiles that cross from one into the next
    (1, 536, 2, 2, 1, 4, True, True),               # runs of 67 positions inside a 16-row tile, rows past the last
])
def test_fp32_rows_of_a_workgroup(usp, bs, L, hc, hk, hs, U, R, causal, zigzag):
    """Both sides of the line between 16 and 32 rows per workgroup, and the remainders of 16 rows."""
    prob = tl.Problem(990 + L, bs, L, hc, hk, hs, U, R, causal, zigzag, tl.FP32)
    o, lse = _run_usp_fwd(usp, prob)
    ref_o, tol = _check_against_reference(prob, o, lse)
    for rank in range(prob.N):
        assert tl.max_abs(o[rank], ref_o[rank]) <= tol, rank


@pytest.mark.parametrize("hs", [64, 128])
def test_fp32_rank_alone_and_among_all(usp, hs):
    """A rank's workgroups have 16 rows where it runs alone (64 of 32 rows) and 32 among all four (256): its rows are summed in
    another order.  Each sum is within the oracle test's tolerance of the exact one, so the two are within twice that."""
    prob = tl.Problem(960 + hs, 1, 1024, 8, 8, hs, 1, 4, False, True, tl.FP32)
    o, lse = _run_usp_fwd(usp, prob)
    o1, lse1 = _run_usp_fwd(usp, prob, 2, 3)
    assert tl.max_abs(o[2], o1[2]) <= 2 * 2e-5 and tl.max_abs(lse[2], lse1[2]) <= 2 * 2e-5
    ref_o, tol = _check_against_reference(prob, o1, lse1, ranks=[2])
    assert tl.max_abs(o1[2], ref_o[2]) <= tol


def test_a_rank_range_writes_only_its_slices(usp):
    """bs = 2, ranks 1 and 2 of four: their head slices, everything else as it was; the other ranks' LSE too."""
    prob = tl.Problem(951, 2, 160, 4, 2, 64, 2, 2, True, True, tl.FP32)
    o, lse = _run_usp_fwd(usp, prob, 1, 3)
    ref_o, tol = _check_against_reference(prob, o, lse, ranks=[1, 2])
    assert np.isnan(lse[0]).all() and np.isnan(lse[3]).all()
    for shard in range(4):      # rank 1 = (r 0, u 1): heads 2, 3 of shards 0, 1; rank 2 = (r 1, u 0): heads 0, 1 of shards 2, 3
        mine = slice(2, 4) if shard < 2 else slice(0, 2)
        other = slice(0, 2) if shard < 2 else slice(2, 4)
        assert tl.max_abs(o[shard][:, :, mine], ref_o[shard][:, :, mine]) <= tol
        assert np.isnan(o[shard][:, :, other]).all()


@pytest.mark.parametrize("o_dtype", [tl.FP32, tl.BF16])
@pytest.mark.parametrize("case", BLOCK_CASES, ids=[c[0] for c in BLOCK_CASES])
def test_block_step_fp32_every_mask(usp, case, o_dtype):
    _, bs, Lq, Lk, hq, hkv, hs, causal, qd, kd = case
    qd, kd = (_desc(usp, *d) if d else None for d in (qd, kd))
    o, lse, ref_o, ref_l = _run_block(usp, 77, bs, Lq, Lk, hq, hkv, hs, causal, qd, kd, tl.FP32, o_dtype)
    tl.assert_lse_close(lse, ref_l, 2e-5)
    assert tl.max_abs(o, ref_o) <= (2e-5 if o_dtype == tl.FP32 else 2e-2)


@pytest.mark.parametrize("hs", [64, 128])
@pytest.mark.parametrize("blocks", [[64, 1500, 100, 1500], [1500, 64], [1500], [33, 1], [1400, 1400, 7]])
def test_state_passes_between_the_kernels(usp, blocks, hs):
    """A ring whose calls are short and long in turn: the 256-row kernel and this one take up each other's running state
    (same records).  Against double precision: weights and O rounded to bf16, below 2^-7."""
    Lq, hq, hkv = 1000, 16, 8
    gen = torch.Generator(device="cuda").manual_seed(len(blocks))
    q = torch.randn((1, Lq, hq, hs), generator=gen, device="cuda", dtype=torch.bfloat16)
    kv = [[torch.randn((1, n, hkv, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for n in blocks] for _ in range(2)]
    state = torch.full((usp.usp_block_attn_fwd_state_bytes(1, Lq, hq, hs),), 0xFF, dtype=torch.uint8, device="cuda")
    o = torch.zeros_like(q)
    lse = torch.zeros((1, hq, Lq), device="cuda")
    for i, n in enumerate(blocks):
        usp.usp_block_attn_fwd_state(q, kv[0][i], kv[1][i], state, o, lse, 1, Lq, n, hq, hkv, hs, 0.0, False, None, None,
                                     i == 0, i == len(blocks) - 1, usp.USP_BF16)
    k, v = (torch.cat([x[0] for x in t]).double().repeat_interleave(hq // hkv, 1) for t in kv)
    for h in range(hq):
        s = q[0, :, h].double() @ k[:, h].T * hs ** -0.5
        ref = s.softmax(-1) @ v[:, h]
        assert ((o[0, :, h].double() - ref).norm() / ref.norm()).item() < 2 ** -7
        assert (lse[0, h].double() - s.logsumexp(-1)).abs().max().item() < 1e-4


def _shifted(t):
    """The same values one element past a multiple of 16 bytes."""
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)
    return buf[1:1 + t.numel()].view(t.shape).copy_(t)


@pytest.mark.parametrize("hs", [64, 128])
@pytest.mark.parametrize("dtype", [tl.BF16, tl.FP32], ids=["bf16", "fp32"])
def test_tensors_may_begin_at_any_element(usp, dtype, hs):
    """Bitwise the same results: one block on dense tensors, and (fp32; bf16 tensors like these are staged for other kernels)
    all ranks of a batch of two whose tiles cross from shard to shard."""
    torch_dtype = torch.float32 if dtype == tl.FP32 else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(hs)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch_dtype)

    q, k, v = normal(2, 100, 4, hs), normal(2, 150, 2, hs), normal(2, 150, 2, hs)
    results = []
    for place in (torch.clone, _shifted):
        o, lse = place(torch.zeros_like(q)), torch.zeros((2, 4, 100), device="cuda")
        usp.usp_block_attn_fwd(place(q), place(k), place(v), o, lse, 2, 100, 150, 4, 2, hs, 0.0, False, None, None, dtype, dtype)
        results.append((o, lse))
    assert all(torch.equal(x, y) for x, y in zip(*results))
    if dtype == tl.BF16:
        return
    p = usp.problem(2, 264, 4, 2, hs, 2, 2, True, usp.USP_SPLIT_ZIGZAG, usp.USP_FP32)
    q, k, v = normal(4, 2, 66, 4, hs), normal(4, 2, 66, 2, hs), normal(4, 2, 66, 2, hs)
    ws = torch.empty(usp.usp_attn_fwd_workspace_bytes(p, 4), dtype=torch.uint8, device="cuda")
    results = []
    for place in (torch.clone, _shifted):
        o, lse = place(torch.zeros_like(q)), torch.zeros((4, 2, 2, 132), device="cuda")
        usp.usp_attn_fwd(p, place(q), place(k), place(v), o, lse, 0, 4, ws)
        results.append((o, lse))
    assert all(torch.equal(x, y) for x, y in zip(*results))
