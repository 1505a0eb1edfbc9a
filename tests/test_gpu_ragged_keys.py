"""The last tile of keys where it is not a whole one: nothing behind the last row of K and V gets into the results.  K and V
lie at the start of a larger buffer that is NaN from there on, and results are compared bit for bit with tensors of their
own, behind which nothing is chosen."""
import pytest
import torch

import paper_2405_07719_amd as usp

pytestmark = pytest.mark.gpu


def nan_behind(t):
    """The same values, 64 rows of NaN behind the last of them."""
    buf = torch.full((t.numel() + 64 * t.shape[-2] * t.shape[-1],), float("nan"), dtype=t.dtype, device=t.device)
    return buf[:t.numel()].view(t.shape).copy_(t)


@pytest.mark.parametrize("dtype", [usp.USP_BF16, usp.USP_FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("hs", [64, 128])
@pytest.mark.parametrize("Lk", [1, 5, 31, 33, 69, 255, 261])     # one to eight waves with a tile; 1, 5 and 31 keys in the last
@pytest.mark.parametrize("causal", [False, True])
def test_nothing_behind_the_last_key_is_used(Lk, hs, dtype, causal):
    bs, hq, hkv, Lq = 2, 4, 2, 40
    torch_dtype = torch.bfloat16 if dtype == usp.USP_BF16 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(Lk)
    q = torch.randn((bs, Lq, hq, hs), generator=gen, device="cuda", dtype=torch_dtype)
    k, v = (torch.randn((bs, Lk, hkv, hs), generator=gen, device="cuda", dtype=torch_dtype) for _ in range(2))
    qpos, kpos = (usp.usp_posdesc(Lk // 2, Lq, 0, 0), usp.usp_posdesc(0, Lk, 0, 0)) if causal else (None, None)

    def step(k, v):
        o = torch.zeros((bs, Lq, hq, hs), device="cuda", dtype=torch_dtype)
        lse = torch.zeros((bs, hq, Lq), device="cuda")
        usp.usp_block_attn_fwd(q, k, v, o, lse, bs, Lq, Lk, hq, hkv, hs, 0.0, causal, qpos, kpos, dtype, dtype)
        out = [o, lse]
        if dtype == usp.USP_BF16:
            state = torch.zeros(usp.usp_block_attn_fwd_state_bytes(bs, Lq, hq, hs), dtype=torch.uint8, device="cuda")
            o, lse = torch.zeros_like(o), torch.zeros_like(lse)
            usp.usp_block_attn_fwd_state(q, k, v, state, o, lse, bs, Lq, Lk, hq, hkv, hs, 0.0, causal, qpos, kpos, True, True, dtype)
            out += [o, lse]
        # the whole forward of one rank
        p = usp.problem(bs, Lk, hkv, hkv, hs, 1, 1, causal, usp.USP_SPLIT_CONTIG, dtype)
        ws = torch.empty(max(256, usp.usp_attn_fwd_workspace_bytes(p, 1)), dtype=torch.uint8, device="cuda")
        o, lse = torch.zeros((1, *k.shape), device="cuda", dtype=torch_dtype), torch.zeros((1, bs, hkv, Lk), device="cuda")
        usp.usp_attn_fwd(p, q_self, k, v, o, lse, 0, 1, ws)
        return out + [o, lse]

    q_self = torch.randn((1, bs, Lk, hkv, hs), generator=gen, device="cuda", dtype=torch_dtype)
    for x, y in zip(step(nan_behind(k), nan_behind(v)), step(k, v)):
        assert torch.isfinite(x.float()).all() and torch.equal(x, y)
