"""Forwards without a mask whose last query tiles are cut into more than four pieces of the keys, up to the eight that a merge
takes, with lengths that end inside a tile: the routes on the CPU, the results against double precision."""
import pytest
import torch

import paper_2405_07719_amd as usp
from tests.host_side import HostSide, problem

# L, query heads, KV heads, head size, Ulysses degree; pieces
SHAPES = [((4368, 16, 8, 128, 1), 5), ((4600, 16, 8, 128, 1), 6), ((8850, 8, 8, 64, 1), 7), ((9000, 16, 4, 128, 2), 8)]


def test_routes(tmp_path):
    host = HostSide(tmp_path)
    for (L, hc, hk, hs, U), pieces in SHAPES:
        route = host.forward(problem(1, L, hc, hk, hs, U, 1, causal=False), 0, 1)
        assert route["kind"] == "listed" and route["parts"] == pieces, (L, route)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [s for s, _ in SHAPES], ids=str)
def test_against_double_precision(shape):
    L, hc, hk, hs, U = shape
    gen = torch.Generator(device="cuda").manual_seed(L)
    q = torch.randn((U, 1, L // U, hc, hs), generator=gen, device="cuda", dtype=torch.bfloat16)
    k, v = (torch.randn((U, 1, L // U, hk, hs), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    p = usp.problem(1, L, hc, hk, hs, U, 1, False, usp.USP_SPLIT_CONTIG, usp.USP_BF16)
    ws = torch.full((usp.usp_attn_fwd_workspace_bytes(p, 1),), 255, dtype=torch.uint8, device="cuda")
    o, lse = torch.full_like(q, float("nan")), torch.full((U, 1, hc // U, L), float("nan"), device="cuda")
    for rank in range(U):
        usp.usp_attn_fwd(p, q, k, v, o, lse, rank, rank + 1, ws)
    qd, kd, vd, od = (x.transpose(0, 1).reshape(L, -1, hs) for x in (q, k, v, o))
    for h in range(0, hc, 3):
        s = qd[:, h].double() @ kd[:, h // (hc // hk)].double().T * hs ** -0.5
        ref = s.softmax(-1) @ vd[:, h // (hc // hk)].double()
        # weights and O rounded to bf16, 2^-9 relative each; the log-sum-exp in fp32: a rounding of some 10 of each of its parts
        assert ((od[:, h].double() - ref).norm() / ref.norm()).item() < 2 ** -7
        assert (lse[h // (hc // U), 0, h % (hc // U)].double() - s.logsumexp(-1)).abs().max().item() < 1e-5
