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


def test_backward_of_some_ranks_of_a_long_batch():
    """2^33 + 2^18 elements of dK and as many of dV, from fp32 accumulators (two of three ranks add to them) in one
    conversion of four elements to a thread: just above 2^32 threads.  Q is its own O and dO, K its own V."""
    room(165)
    bs, L, heads, hs, R = 10923, 192, 32, 128, 3
    assert 2 * bs * L * heads * hs // 4 > 2 ** 32
    p = usp.problem(bs, L, heads, heads, hs, 1, R, False, usp.USP_SPLIT_CONTIG, usp.USP_BF16)
    shape = (R, bs, L // R, heads, hs)
    q, k = (torch.zeros(shape, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    gen = torch.Generator(device="cuda").manual_seed(4)
    entries = [0, 1, bs // 2, bs - 2, bs - 1]
    for t in (q, k):
        for b in entries:
            t[:, b] = torch.randn(t[:, b].shape, generator=gen, device="cuda", dtype=torch.float32)
    lse = torch.full((R, bs, heads, L // R), 6.0, device="cuda")     # any value will do: P = exp(s - LSE)
    dq = torch.empty_like(q)
    dk, dv = (torch.full_like(k, float("nan")) for _ in range(2))
    ws = torch.empty(usp.usp_attn_bwd_workspace_bytes(p, 2), dtype=torch.uint8, device="cuda")
    usp.usp_attn_bwd(p, q, k, k, q, lse, q, dq, dk, dv, 0, 2, ws)
    scale = hs ** -0.5
    for b in entries:
        kd = k[:, b].reshape(L, heads, hs).double().cpu()
        qd = q[:2, b].reshape(2 * L // R, heads, hs).double().cpu()   # the rows of ranks 0 and 1
        w = torch.exp(torch.einsum("qhe,khe->hqk", qd, kd) * scale - 6.0)
        ds = w * (torch.einsum("qhe,khe->hqk", qd, kd) - (qd * qd).sum(-1).T[:, :, None])
        for got, want in ((dk, torch.einsum("hqk,qhe->khe", ds, qd) * scale), (dv, torch.einsum("hqk,qhe->khe", w, qd))):
            x = got[:, b].reshape(L, heads, hs).double().cpu()
            assert (x - want).norm() / want.norm() < 2 ** -7          # P, dS and the result rounded to bf16
        x, want = dq[:2, b].reshape(2 * L // R, heads, hs).double().cpu(), torch.einsum("hqk,khe->qhe", ds, kd) * scale
        assert (x - want).norm() / want.norm() < 2 ** -7
    others = torch.ones(bs, dtype=torch.bool)
    others[entries] = False
    for b in others.nonzero()[::97, 0].tolist():
        assert dk[:, b].abs().max() == 0 and dv[:, b].abs().max() == 0
