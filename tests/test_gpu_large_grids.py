"""Problems with more threads than one launch may have: a long batch of short sequences, tens of GiB.  Some batch entries at
the ends of the batch and around the place where the second launch takes over hold random values and are checked in double
precision; all others are zeros, whose outputs are zeros."""
import pytest
import torch

import paper_2405_07719_amd as usp

pytestmark = pytest.mark.gpu


def room(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib * 2 ** 30:
        pytest.skip(f"needs {gib} GiB of GPU memory")


def attention(q, k, v, causal):
    """[L, heads, hs] tensors in double precision -> O, LSE."""
    q, k, v = (t.double() for t in (q, k, v))
    k, v = (t.repeat_interleave(q.shape[1] // t.shape[1], 1) for t in (k, v))
    s = torch.einsum("qhe,khe->hqk", q.cpu(), k.cpu()) * q.shape[-1] ** -0.5
    if causal:
        s = s.masked_fill(torch.ones(s.shape[-2:]).triu(1).bool(), float("-inf"))
    return torch.einsum("hqk,khe->qhe", s.softmax(-1), v.cpu()), s.logsumexp(-1)


def test_fp32_forward_of_a_long_batch():
    """270 million rows of a head, 512 threads for every 32 of them: just above 2^32 threads.  O over Q, to halve the room."""
    room(100)
    bs, L, hc, hk, hs, U = 4000, 128, 528, 8, 64, 8
    assert bs * L * hc // 32 * 512 > 2 ** 32
    p = usp.problem(bs, L, hc, hk, hs, U, 1, True, usp.USP_SPLIT_CONTIG, usp.USP_FP32)
    q = torch.zeros((U, bs, L // U, hc, hs), device="cuda")
    k, v = (torch.zeros((U, bs, L // U, hk, hs), device="cuda") for _ in range(2))
    gen = torch.Generator(device="cuda").manual_seed(3)
    wgs_before = 2 ** 32 // 512     # the items are the rows of the last query tile first, batch entries fastest but for heads
    entries = [0, 1, wgs_before // hk % bs, bs // 2, bs - 2, bs - 1]
    for t in (q, k, v):
        for b in entries:
            t[:, b] = torch.randn(t[:, b].shape, generator=gen, device="cuda")
    ref = {b: attention(*(t[:, b].reshape(L, -1, hs) for t in (q, k, v)), True) for b in entries}
    lse = torch.full((U, bs, hc // U, L), float("nan"), device="cuda")
    ws = torch.empty(usp.usp_attn_fwd_workspace_bytes(p, U), dtype=torch.uint8, device="cuda")
    usp.usp_attn_fwd(p, q, k, v, q, lse, 0, U, ws)
    for b in entries:
        o, l = ref[b]
        got = q[:, b].reshape(L, hc, hs).double().cpu()
        assert (got - o).norm() / o.norm() < 3.5e-6      # fp32 sums: as tests at ordinary sizes see, 4e-7 to 8e-7, times four
        assert (lse[:, b].reshape(hc, L).double().cpu() - l).abs().max() < 2e-5
    assert torch.isfinite(lse).all()                     # every row of every entry was written
    others = torch.ones(bs, dtype=torch.bool)
    others[entries] = False
    zero = torch.log(torch.arange(1, L + 1, device="cuda", dtype=torch.float64)).float()
    for b in others.nonzero()[::97, 0].tolist():         # scores of zero: LSE is the log of the number of visible keys
        assert (lse[:, b] - zero).abs().max() < 2e-5 and q[:, b].abs().max() == 0
