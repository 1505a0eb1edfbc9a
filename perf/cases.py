"""The work that a user of this framework has it do, as timed cases.

One case is one call (or one training step, or one ring loop) through the public entry points, on inputs that lie in
HBM.  The listed cases are the five configurations that the benchmark and the parity tests are built on, the shortest
sequence of the paper's attention tables, a bidirectional ragged one, a ring that receives its blocks one per call, and
the all-to-alls alone; `draw` gives further cases of the same kinds, sizes and options.
"""
import math

import torch

import paper_2405_07719_amd as usp

# what the benchmark's configurations share: 32 query heads on 8 KV heads of size 128
_DEFAULTS = {"bs": 1, "hc": 32, "hk": 8, "hs": 128, "causal": True, "zigzag": True, "dtype": "bf16", "rank": 0,
             "all_ranks": False}


def _case(name, kind, L, U, R, **more):
    case = dict(_DEFAULTS, kind=kind, L=L, U=U, R=R, **more)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the tiny check in single precision: every rank of Ulysses 2 x ring 2, where launches and latency are all there is
        _case("fwd_tiny_fp32", "forward", 256, 2, 2, hc=4, hk=4, hs=64, causal=False, zigzag=False, dtype="fp32",
              all_ranks=True),
        # a short prompt on every rank of a small group (the size of the smoke check): latency again, in bf16
        _case("fwd_short_all_ranks", "forward", 1024, 2, 2, hc=8, hk=4, all_ranks=True),
        # the shortest sequence of the paper's attention tables on one Ulysses rank: too few query tiles to fill the chip
        _case("fwd_L8192_u8", "forward", 8192, 8, 1),
        # the ordinary size: the Ulysses-only rank, and the ring-only rank, of L = 32768
        _case("fwd_L32768_u8", "forward", 32768, 8, 1),
        _case("fwd_L32768_ring8", "forward", 32768, 1, 8),
        # the largest: one rank of Ulysses 8 x ring 2 at 208K tokens (the benchmark's default workload)
        _case("fwd_L212992_u8r2", "forward", 212992, 8, 2),
        # visual tokens, attended both ways: no mask, as many KV heads as query heads, head size 64, a ragged length
        _case("fwd_bidirectional_hs64_ragged", "forward", 17776, 8, 1, hk=32, hs=64, causal=False),
        # a ring whose blocks arrive one per step: eight calls that carry the running softmax state
        _case("ring_steps_L32768", "ring_steps", 32768, 1, 8, steps="state"),
        # the backward of a short sequence, and of the ordinary one, with the plain workspace
        _case("bwd_L8192_u8", "backward", 8192, 8, 1, keep_ds=False),
        _case("bwd_L32768_u8", "backward", 32768, 8, 1, keep_ds=False),
        # a training step of one rank of Ulysses 2 x ring 4: forward, then backward with the workspace that keeps dS
        _case("train_L65536_u2r4", "train", 65536, 2, 4, keep_ds=True),
        # Algorithm 1's all-to-alls alone, all ranks: Q, K, V to head layout, O back
        _case("layout_L32768_u8", "layout", 32768, 8, 1, all_ranks=True),
    ]


# ---------------------------------------------------------------------------------------------------------------
# drawn cases
# ---------------------------------------------------------------------------------------------------------------
_GROUPS = [(8, 1), (4, 2), (2, 4), (1, 8), (8, 2), (2, 2), (1, 4), (4, 1), (1, 1), (2, 1), (1, 2)]


def _length(rng, lo, hi, unit):
    """A sequence length in [lo, hi], even over its logarithm, that the ranks can share (a multiple of `unit`)."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(unit, int(x / unit) * unit)


def draw(rng):
    kind = rng.choices(["forward", "fp32", "ring_steps", "backward", "train", "layout"], [40, 10, 12, 18, 8, 12])[0]
    U, R = rng.choice(_GROUPS)
    hc, hk = rng.choice([(32, 8), (32, 8), (32, 32), (16, 8), (32, 1)])
    if hk == 1:                      # one KV head: the ring alone can split the sequence
        U = 1
    hs = rng.choice([128, 128, 128, 64])
    causal = rng.random() < 0.75
    zigzag = rng.random() < 0.8
    unit = 2 * U * R
    rank = rng.randrange(U * R)
    if kind == "fp32":
        hc, hk = rng.choice([(4, 4), (8, 4), (4, 2)])
        U, R = rng.choice([(2, 2), (1, 4), (2, 1), (1, 1), (1, 2)])
        return _case(None, "forward", _length(rng, 128, 2048, 2 * U * R), U, R, hc=hc, hk=hk, hs=hs, causal=causal,
                     zigzag=zigzag, dtype="fp32", all_ranks=True, bs=rng.choice([1, 1, 2]))
    if kind == "layout":
        return _case(None, kind, _length(rng, 1024, 131072, unit), U, R, hc=hc, hk=hk, hs=hs, zigzag=zigzag,
                     all_ranks=True)
    lo, hi = {"forward": (512, 212992), "ring_steps": (2048, 65536), "backward": (1024, 65536), "train": (1024, 65536)}[kind]
    if kind == "ring_steps":
        U, R = rng.choice([(1, 8), (2, 4), (4, 2), (1, 4), (1, 2)]) if hk > 1 else (1, rng.choice([2, 4, 8]))
        unit, rank = 2 * U * R, rng.randrange(U * R)
    bound = {"forward": 2.0e13, "ring_steps": 5.0e12, "backward": 1.0e13, "train": 1.4e13}[kind]
    while True:
        L = _length(rng, lo, hi, unit)
        case = _case(None, kind, L, U, R, hc=hc, hk=hk, hs=hs, causal=causal, zigzag=zigzag, rank=rank,
                     bs=rng.choice([1, 1, 2]) if L <= 16384 else 1)
        if kind == "ring_steps":
            case["steps"] = rng.choice(["state", "partials"])
        if kind in ("backward", "train"):
            case["keep_ds"] = rng.random() < 0.4 and L <= 65536 and _pairs_all(case) * 2 < 40e9
        case["all_ranks"] = kind != "ring_steps" and L <= 4096 and rng.random() < 0.5
        if work(case)["flops"] <= bound:
            return case


# ---------------------------------------------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------------------------------------------
def _ranks(case):
    return (0, case["U"] * case["R"]) if case["all_ranks"] else (case["rank"], case["rank"] + 1)


def _problem(case):
    return usp.problem(case["bs"], case["L"], case["hc"], case["hk"], case["hs"], case["U"], case["R"], case["causal"],
                       usp.USP_SPLIT_ZIGZAG if case["zigzag"] else usp.USP_SPLIT_CONTIG,
                       usp.USP_FP32 if case["dtype"] == "fp32" else usp.USP_BF16)


def _runs(case, ring_rank):
    """The ascending runs (first position, length) of a ring rank's rows: two chunks of 2R, or one of R."""
    L, R = case["L"], case["R"]
    if case["zigzag"]:
        c = L // (2 * R)
        return [(ring_rank * c, c), ((2 * R - 1 - ring_rank) * c, c)]
    return [(ring_rank * (L // R), L // R)]


def _pairs(case):
    """(query, key) pairs that the mask lets through, all heads and batches of the ranks that run."""
    total = 0
    for rank in range(*_ranks(case)):
        for start, n in _runs(case, rank // case["U"]):
            total += n * start + n * (n + 1) // 2 if case["causal"] else n * case["L"]
    return total * (case["hc"] // case["U"]) * case["bs"]


def _pairs_all(case):
    """Pairs, masked or not, of one rank: what a kept dS holds."""
    return (case["L"] // case["R"]) * case["L"] * (case["hc"] // case["U"]) * case["bs"]


def work(case):
    es = 4 if case["dtype"] == "fp32" else 2
    U, R, bs, L, hs = case["U"], case["R"], case["bs"], case["L"], case["hs"]
    begin, end = _ranks(case)
    q_rank = bs * (L // R) * (case["hc"] // U) * hs           # elements of Q (and O, dO, dQ) of one rank
    n_cols = len({rank % U for rank in range(begin, end)})
    kv = bs * L * (case["hk"] // U) * hs * n_cols             # elements of K (and V, dK, dV) that the ranks read
    lse = bs * (L // R) * (case["hc"] // U) * 4 * (end - begin)
    q_all = q_rank * (end - begin)
    if case["kind"] == "layout":
        return {"bytes": 2 * es * (2 * q_all + 2 * kv), "flops": 0}
    forward = es * (2 * q_all + 2 * kv) + lse
    backward = es * (4 * q_all + 4 * kv) + lse
    flops = 4 * hs * _pairs(case)
    return {"forward": {"bytes": forward, "flops": flops},
            "ring_steps": {"bytes": forward, "flops": flops},
            "backward": {"bytes": backward, "flops": 2.5 * flops},
            "train": {"bytes": forward + backward, "flops": 3.5 * flops}}[case["kind"]]


# ---------------------------------------------------------------------------------------------------------------
# what a user's program has in hand, and one pass
# ---------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    """Inputs iid N(0,1) in the sequence layout [N][bs][L/N][heads][hs] (a ring of steps: already in head layout)."""
    dtype = torch.float32 if case["dtype"] == "fp32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)

    def bytes_(n):
        return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")

    p = _problem(case)
    bs, U, R, N, L, hs = case["bs"], case["U"], case["R"], case["U"] * case["R"], case["L"], case["hs"]
    hq, hkv, Lq = case["hc"] // U, case["hk"] // U, L // R
    begin, end = _ranks(case)
    s = {"case": case, "p": p}
    if case["kind"] == "ring_steps":
        r, u = divmod(case["rank"], U)
        s["q"] = normal(bs, Lq, hq, hs)
        s["k"] = [normal(bs, Lq, hkv, hs) for _ in range(R)]
        s["v"] = [normal(bs, Lq, hkv, hs) for _ in range(R)]
        s["qpos"] = usp.usp_local_positions(p, r, u)[1]
        s["kpos"] = [usp.usp_local_positions(p, (r - i) % R, u)[1] for i in range(R)]
        s["o"] = torch.zeros(bs, Lq, hq, hs, device="cuda", dtype=dtype)
        s["lse"] = torch.zeros(bs, hq, Lq, device="cuda")
        if case["steps"] == "state":
            s["state"] = bytes_(usp.usp_block_attn_fwd_state_bytes(bs, Lq, hq, hs))
        else:
            s["o_parts"] = [torch.empty(bs, Lq, hq, hs, device="cuda") for _ in range(R)]
            s["lse_parts"] = [torch.empty(bs, hq, Lq, device="cuda") for _ in range(R)]
        return s
    q_shape, kv_shape = (N, bs, L // N, case["hc"], hs), (N, bs, L // N, case["hk"], hs)
    s["q"], s["k"], s["v"] = normal(*q_shape), normal(*kv_shape), normal(*kv_shape)
    if case["kind"] == "layout":
        s["o_head"] = normal(N, bs, Lq, hq, hs)
        s["o"] = torch.zeros_like(s["q"])
        s["q_head"] = torch.zeros_like(s["o_head"])
        s["k_head"] = torch.zeros(N, bs, Lq, hkv, hs, device="cuda", dtype=dtype)
        s["v_head"] = torch.zeros_like(s["k_head"])
        return s
    s["o"] = torch.zeros_like(s["q"])
    s["lse"] = torch.zeros(N, bs, hq, Lq, device="cuda")
    s["ws"] = bytes_(usp.usp_attn_fwd_workspace_bytes(p, end - begin))
    if case["kind"] in ("backward", "train"):
        need = usp.usp_attn_bwd_workspace_bytes_with_ds if case["keep_ds"] else usp.usp_attn_bwd_workspace_bytes
        s["ws_bwd"] = bytes_(need(p, end - begin))
        s["do"] = normal(*q_shape)
        s["dq"], s["dk"], s["dv"] = torch.zeros_like(s["q"]), torch.zeros_like(s["k"]), torch.zeros_like(s["v"])
        if case["kind"] == "backward":       # O and LSE come from the forward, which ran earlier in the step
            usp.usp_attn_fwd(p, s["q"], s["k"], s["v"], s["o"], s["lse"], begin, end, s["ws"])
    return s


def run(s):
    case, p = s["case"], s["p"]
    begin, end = _ranks(case)
    kind = case["kind"]
    if kind == "layout":
        usp.usp_layout_a2a(p, case["hc"], usp.USP_SEQ_TO_HEAD, s["q"], s["q_head"], begin, end)
        usp.usp_layout_a2a(p, case["hk"], usp.USP_SEQ_TO_HEAD, s["k"], s["k_head"], begin, end)
        usp.usp_layout_a2a(p, case["hk"], usp.USP_SEQ_TO_HEAD, s["v"], s["v_head"], begin, end)
        usp.usp_layout_a2a(p, case["hc"], usp.USP_HEAD_TO_SEQ, s["o_head"], s["o"], begin, end)
        return {"q_head": s["q_head"], "k_head": s["k_head"], "v_head": s["v_head"], "o": s["o"]}
    if kind == "ring_steps":
        R, bs, hs = case["R"], case["bs"], case["hs"]
        hq, hkv, Lq, causal = case["hc"] // case["U"], case["hk"] // case["U"], case["L"] // case["R"], case["causal"]
        for i in range(R):
            if case["steps"] == "state":
                usp.usp_block_attn_fwd_state(s["q"], s["k"][i], s["v"][i], s["state"], s["o"], s["lse"], bs, Lq, Lq, hq, hkv,
                                             hs, 0.0, causal, s["qpos"], s["kpos"][i], i == 0, i == R - 1, usp.USP_BF16)
            else:
                usp.usp_block_attn_fwd(s["q"], s["k"][i], s["v"][i], s["o_parts"][i], s["lse_parts"][i], bs, Lq, Lq, hq, hkv,
                                       hs, 0.0, causal, s["qpos"], s["kpos"][i], usp.USP_BF16, usp.USP_FP32)
        if case["steps"] == "partials":
            usp.usp_lse_merge(s["o_parts"], s["lse_parts"], s["o"], s["lse"], bs, Lq, hq, hs, usp.USP_FP32, usp.USP_BF16)
        return {"o": s["o"], "lse": s["lse"]}
    out = {}
    if kind in ("forward", "train"):
        usp.usp_attn_fwd(p, s["q"], s["k"], s["v"], s["o"], s["lse"], begin, end, s["ws"])
        out.update(o=s["o"], lse=s["lse"])
    if kind in ("backward", "train"):
        usp.usp_attn_bwd(p, s["q"], s["k"], s["v"], s["o"], s["lse"], s["do"], s["dq"], s["dk"], s["dv"], begin, end,
                         s["ws_bwd"])
        out.update(dq=s["dq"], dk=s["dk"], dv=s["dv"])
    return out


def tolerance(case):
    """Four times what the outputs show against the same attention in double precision, measured over drawn cases of every
    kind: bf16 (P and dS rounded to bf16 for the matrix core, bf16 results) 2.1e-3 to 2.4e-3 on O, dQ, dK and dV, largest
    difference 2.2e-2; fp32 3.7e-7 to 8.0e-7, largest 7.7e-6."""
    if case["kind"] == "layout":
        return "exact"
    if case["dtype"] == "fp32":
        return {"rel": 3.5e-6, "max": 4e-5}
    return {"rel": 1e-2, "max": 0.1}
