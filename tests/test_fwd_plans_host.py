"""How the forward of a rank is cut, on the CPU: which answers are worked out and when, and the launches played through."""
import heapq
import random

import pytest

import paper_2405_07719_amd as usp
from tests.host_side import HostSide, problem
from tests.test_gpu_attn_fwd import CUT, MODEL_SHAPES
from tests.test_gpu_ring import STATE_STEPS


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    return HostSide(tmp_path_factory.mktemp("host_side"))


@pytest.mark.parametrize("heads", [1, 2, 3, 4, 6, 12, 32, 96, 256, 300, 512])
def test_one_workgroup_plays_for_all_alike(host, heads):
    """The end of a launch is that of 256 workgroups, the first one that is free taking the next item, to the last bit: the
    same sums in the same order."""
    rng = random.Random(heads)
    for n in [1, 2, 7, 40, 150]:
        us = [rng.choice([9.0, 10.78, 23.5, rng.uniform(8, 200)]) for _ in range(n)]
        for items in (us, sorted(us, reverse=True)):
            free, end = [0.0] * 256, 0.0
            for x in items:
                for _ in range(heads):
                    done = heapq.heappop(free) + x
                    end = max(end, done)
                    heapq.heappush(free, done)
            assert host.played(heads, items) == end


def test_items_are_listed_for_the_ranks_that_are_launched(host):
    """... and not for a workspace query about several ring ranks, a problem that goes to the one short launch, or ranks that nobody asked for."""
    p = problem(1, 16384, 32, 8, 128, 4, 2)
    assert host.query(p) > 0 and host.ranks_listed(p) == 0
    assert host.forward(p, 5, 6)["kind"] == "listed" and host.ranks_listed(p) == 1
    assert host.forward(p, 6, 7)["kind"] == "listed" and host.ranks_listed(p) == 1      # the same ring rank
    assert host.forward(p, 0, 8)["launches"] == 8 and host.ranks_listed(p) == 2
    one = problem(1, 8192, 32, 8, 128, 8, 1)
    assert host.query(one) > 0 and host.ranks_listed(one) == 1                          # there is no other ring rank
    short = problem(1, 2048, 32, 8, 128, 8, 1)
    assert host.forward(short, 0, 1)["kind"] == "waves" and host.ranks_listed(short) == 0
    many = problem(1, 2 * 17 * 4096, 32, 8, 128, 1, 17)      # more blocks than one launch takes
    assert host.forward(many, 0, 1)["kind"] == "blocks" and host.ranks_listed(many) == 0


def test_answers_are_kept_for_the_last_problems(host):
    """64 of them, whichever were asked about last."""
    kept = problem(1, 16384, 32, 8, 128, 4, 2, zigzag=False)
    assert host.forward(kept, 7, 8)["kind"] == "listed" and host.ranks_listed(kept) == 1
    for i in range(100):
        host.query(problem(1, 6144 + 16 * i, 32, 8, 128, 8, 1))
        assert host.ranks_listed(kept) == 1
    for i in range(64):
        host.query(problem(1, 6144 + 16 * i, 16, 8, 128, 8, 1))
    assert host.ranks_listed(kept) == 0


@pytest.mark.parametrize("dtype", [usp.USP_BF16, usp.USP_FP32])
def test_the_same_launch_every_time(host, dtype):
    for p in [problem(1, 8192, 32, 8, 128, 8, 1, dtype=dtype), problem(2, 4608, 8, 2, 64, 1, 2, dtype=dtype)]:
        first = host.forward(p, 0, 1)
        assert host.forward(p, 0, 1) == first


@pytest.mark.parametrize("case", CUT)
def test_the_gpu_cases_take_their_launch(host, case):
    *shape, rank, causal, zigzag, launch, parts = case
    got = host.forward(problem(*shape, causal, zigzag), rank, rank + 1)
    assert (got["kind"], got["parts"]) == (launch, parts), got


def test_the_gpu_cases_cover_every_cut(host):
    """Lists with and without whole items, parts of the same and of different rows, two to eight parts, one and several batch
    entries; the older cuts that rings of 9 to 16 blocks take."""
    listed = []
    for *shape, rank, causal, zigzag, launch, parts in CUT:
        got = host.forward(problem(*shape, causal, zigzag), rank, rank + 1)
        listed += [(got["parts"], got["whole"] > 0, got["different_rows"], shape[0] > 1, shape[5] > 1)] if launch == "listed" else []
    assert {2, 3, 4, 8} <= {x[0] for x in listed}
    assert {(w, d) for _, w, d, _, _ in listed} == {(False, 0), (False, 1), (True, 0), (True, 1)}
    assert any(b and u and d for _, _, d, b, u in listed)
    assert {c[-2] for c in CUT} == {"waves", "listed", "last tiles cut", "every tile cut", "blocks"}
    shapes = {name: host.forward(problem(*shape, causal=causal), 0, shape[5] * shape[6])["kind"] for name, *shape, causal in MODEL_SHAPES}
    assert {n for n, kind in shapes.items() if kind == "listed"} == {
        "key_split_3_pieces_noncausal", "heavy_tiles_cut_head_size_64", "heavy_tiles_cut_batch_of_two", "heavy_tiles_cut_ring_of_two",
        "heavy_tiles_cut_short_four_pieces", "tiles_cut_noncausal_to_fill_the_last_round"}


@pytest.mark.parametrize("case", STATE_STEPS, ids=[c[0] for c in STATE_STEPS])
def test_the_gpu_state_steps_go_to_256_row_items(host, case):
    """... with as many query tiles that see the block as the case says: rows of 256 in a row, as the state's records are."""
    name, bs, hs, hq, hkv, rows, blocks, tiles = case
    Lq, Lk = rows[1] + rows[3], blocks[0][1] + blocks[0][3]
    assert all(b[1] + b[3] == Lk for b in blocks)
    assert not host.lib.block_goes_to_waves(bs, host.long(Lq), host.long(Lk), hq, hs, 1, usp.USP_BF16)
    q = [rows[0] + i if i < rows[1] else rows[2] + i - rows[1] for i in range(Lq)]
    starts = [min([b[0]] * (b[1] > 0) + [b[2]] * (b[3] > 0)) for b in blocks]
    assert [sum(max(q[t:t + 256]) >= s for t in range(0, Lq, 256)) for s in starts[1:-1]] == tiles


def test_the_gpu_state_steps_cover_every_list():
    """All tiles, some, one, none; an odd number; as many items as CUs, fewer, and more."""
    items, counts = set(), set()
    for name, bs, hs, hq, hkv, rows, blocks, tiles in STATE_STEPS:
        n = -(-(rows[1] + rows[3]) // 256)
        counts |= {"all" if t == n else "none" if t == 0 else "odd" if t % 2 else "even" for t in tiles}
        items |= {(t * hq * bs > 256) - (t * hq * bs < 256) for t in tiles if 0 < t < n}
    assert counts == {"all", "none", "odd", "even"} and items == {-1, 0, 1}
