// C-ABI entry points: host-side validation, Algorithm 2 index arithmetic, and the
// orchestration of Algorithm 1 (all-to-all -> ring loop -> merge -> all-to-all) over kernels.
// No arithmetic of the method runs on the host; every step is a kernel launch.
#include <math.h>

#include <algorithm>
#include <functional>
#include <memory>
#include <mutex>
#include <numeric>
#include <string.h>
#include <vector>

#include "usp_internal.h"

using namespace usp;

// (Entry points below that keep host-side records, of plans and of counter sets, are function-try-blocks: no exception, as of
// host memory that runs out, passes the C boundary.)

extern "C" const char* usp_status_str(int s) {
  switch (s) {
    case USP_OK: return "ok";
    case USP_ERR_NULL: return "null pointer";
    case USP_ERR_SHAPE: return "bad shape (sizes must be positive; L must divide by N, or by 2*R*U for the zigzag split)";
    case USP_ERR_DEGREE: return "bad degree (need U,R >= 1, hc % U == 0, hk % U == 0, hc % hk == 0)";
    case USP_ERR_DTYPE: return "bad dtype";
    case USP_ERR_WORKSPACE: return "workspace missing or too small";
    case USP_ERR_UNSUPPORTED: return "unsupported configuration";
    case USP_ERR_LAUNCH: return "HIP launch error (or host memory ran out)";
    default: return "unknown status";
  }
}

extern "C" int usp_validate(const usp_problem* p) {
  if (!p) return USP_ERR_NULL;
  if (p->bs < 1 || p->L < 1 || p->hc < 1 || p->hk < 1 || p->hs < 1) return USP_ERR_SHAPE;
  if (p->ulysses < 1 || p->ring < 1) return USP_ERR_DEGREE;
  if (p->hc % p->hk) return USP_ERR_DEGREE;
  // Sec. 3: the Ulysses degree is limited by the (KV) head count.
  if (p->hc % p->ulysses || p->hk % p->ulysses) return USP_ERR_DEGREE;
  if (p->dtype != USP_BF16 && p->dtype != USP_FP32) return USP_ERR_DTYPE;
  if (p->split != USP_SPLIT_CONTIG && p->split != USP_SPLIT_ZIGZAG) return USP_ERR_UNSUPPORTED;
  const int64_t n = (int64_t)p->ulysses * p->ring;
  if (p->split == USP_SPLIT_ZIGZAG) {
    if (p->L % (2 * n)) return USP_ERR_SHAPE;
  } else if (p->L % n) {
    return USP_ERR_SHAPE;
  }
  if (p->hs != 64 && p->hs != 128) return USP_ERR_UNSUPPORTED;
  if (p->L >= (int64_t)1 << 31) return USP_ERR_UNSUPPORTED;
  if (!(p->scale >= 0.0f) || isinf(p->scale)) return USP_ERR_UNSUPPORTED;
  return USP_OK;
}

// Algorithm 2: ring rank r owns chunks r and 2R-1-r (of 2R); Ulysses rank u the u-th of U pieces.
static void ring_block_desc(const usp_problem& p, int r, usp_posdesc* d) {
  if (p.split == USP_SPLIT_ZIGZAG) {
    const int64_t c = p.L / (2 * (int64_t)p.ring);
    d->start0 = (int64_t)r * c;
    d->len0 = c;
    d->start1 = (2 * (int64_t)p.ring - 1 - r) * c;
    d->len1 = c;
  } else {
    const int64_t n = p.L / p.ring;
    d->start0 = (int64_t)r * n;
    d->len0 = n;
    d->start1 = d->start0 + n;
    d->len1 = 0;
  }
}

extern "C" int usp_local_positions(const usp_problem* p, int ring_rank, int ulysses_rank, usp_posdesc* shard,
                                   usp_posdesc* ring_block) {
  int st = usp_validate(p);
  if (st != USP_OK) return st;
  if (ring_rank < 0 || ring_rank >= p->ring || ulysses_rank < 0 || ulysses_rank >= p->ulysses)
    return USP_ERR_UNSUPPORTED;
  usp_posdesc blk;
  ring_block_desc(*p, ring_rank, &blk);
  if (ring_block) *ring_block = blk;
  if (shard) {
    // local indices [a, b) of the ring block, cut against the block's two runs
    const int64_t n = (blk.len0 + blk.len1) / p->ulysses;
    const int64_t a = (int64_t)ulysses_rank * n, b = a + n;
    const int64_t a0 = a < blk.len0 ? a : blk.len0, b0 = b < blk.len0 ? b : blk.len0;   // part in run 0
    const int64_t a1 = (a > blk.len0 ? a : blk.len0) - blk.len0, b1 = (b > blk.len0 ? b : blk.len0) - blk.len0;
    shard->start0 = blk.start0 + a0;
    shard->len0 = b0 - a0;
    shard->start1 = blk.start1 + a1;
    shard->len1 = b1 - a1;
  }
  return USP_OK;
}

extern "C" int usp_layout_a2a(const usp_problem* p, int heads, int dir, const void* src, void* dst, int rank_begin,
                              int rank_end, void* stream) {
  int st = usp_validate(p);
  if (st != USP_OK) return st;
  if (!src || !dst) return USP_ERR_NULL;
  if (heads < 1 || heads % p->ulysses) return USP_ERR_DEGREE;
  if (dir != USP_SEQ_TO_HEAD && dir != USP_HEAD_TO_SEQ && dir != USP_SEQ_TO_HEAD_VT) return USP_ERR_UNSUPPORTED;
  const int n = p->ulysses * p->ring;
  if (rank_begin < 0 || rank_end > n || rank_begin > rank_end) return USP_ERR_UNSUPPORTED;
  if (dir == USP_SEQ_TO_HEAD_VT && p->dtype != USP_BF16) return USP_ERR_DTYPE;
  if (rank_begin == rank_end) return USP_OK;
  if (dir == USP_SEQ_TO_HEAD_VT)
    return launch_layout_a2a_vt(*p, heads, src, dst, rank_begin, rank_end, 0, (hipStream_t)stream);
  return launch_layout_a2a(*p, heads, dir, src, dst, rank_begin, rank_end, 0, (hipStream_t)stream);
}

// Whether na bytes at a and nb bytes at b share memory.
static bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  return (const char*)a < (const char*)b + nb && (const char*)b < (const char*)a + na;
}

static bool desc_ok(const usp_posdesc* d, int64_t len) {
  // positions must fit 32 bits: the kernels narrow them
  const int64_t lim = (int64_t)1 << 31;
  return d && d->len0 >= 0 && d->len1 >= 0 && d->len0 + d->len1 == len && d->start0 >= 0 && d->start1 >= 0 &&
         d->start0 + d->len0 < lim && d->start1 + d->len1 < lim;
}

extern "C" int usp_block_attn_fwd(const void* q, const void* k, const void* v, void* o_part, float* lse_part, int bs,
                                  int64_t Lq, int64_t Lk, int hq, int hkv, int hs, float scale, int causal,
                                  const usp_posdesc* qpos, const usp_posdesc* kpos, int in_dtype, int o_dtype,
                                  void* stream) try {
  if (!q || !k || !v || !o_part || !lse_part) return USP_ERR_NULL;
  if (bs < 1 || Lq < 1 || Lk < 1 || hq < 1 || hkv < 1) return USP_ERR_SHAPE;
  if (hq % hkv) return USP_ERR_DEGREE;
  if (hs != 64 && hs != 128) return USP_ERR_UNSUPPORTED;
  if ((in_dtype != USP_BF16 && in_dtype != USP_FP32) || (o_dtype != USP_BF16 && o_dtype != USP_FP32))
    return USP_ERR_DTYPE;
  if (!(scale >= 0.0f) || isinf(scale)) return USP_ERR_UNSUPPORTED;
  if (Lq >= (int64_t)1 << 31 || Lk >= (int64_t)1 << 31) return USP_ERR_UNSUPPORTED;
  usp_posdesc qd = {0, Lq, 0, 0}, kd = {0, Lk, 0, 0};
  if (causal) {
    if (!qpos || !kpos) return USP_ERR_NULL;
    if (!desc_ok(qpos, Lq) || !desc_ok(kpos, Lk)) return USP_ERR_SHAPE;
    qd = *qpos;
    kd = *kpos;
  }
  if (scale == 0.0f) scale = 1.0f / sqrtf((float)hs);
  return launch_block_attn_fwd(q, k, v, o_part, lse_part, bs, Lq, Lk, hq, hkv, hs, scale, causal ? 1 : 0, qd, kd,
                               in_dtype, o_dtype, (hipStream_t)stream);
} catch (...) {
  return USP_ERR_LAUNCH;
}

extern "C" size_t usp_block_attn_fwd_state_bytes(int bs, int64_t Lq, int hq, int hs) {
  if (bs < 1 || Lq < 1 || hq < 1 || (hs != 64 && hs != 128) || Lq >= (int64_t)1 << 31) return 0;
  return attn_fwd_state_bytes(bs, Lq, hq, hs);
}

extern "C" int usp_block_attn_fwd_state(const void* q, const void* k, const void* v, void* state, size_t state_bytes,
                                        void* o, float* lse, int bs, int64_t Lq, int64_t Lk, int hq, int hkv, int hs,
                                        float scale, int causal, const usp_posdesc* qpos, const usp_posdesc* kpos,
                                        int first, int last, int o_dtype, void* stream) try {
  if (!q || !k || !v || !state) return USP_ERR_NULL;
  if (last && (!o || !lse)) return USP_ERR_NULL;
  if (bs < 1 || Lq < 1 || Lk < 1 || hq < 1 || hkv < 1) return USP_ERR_SHAPE;
  if (hq % hkv) return USP_ERR_DEGREE;
  if (hs != 64 && hs != 128) return USP_ERR_UNSUPPORTED;
  if (o_dtype != USP_BF16 && o_dtype != USP_FP32) return USP_ERR_DTYPE;
  if (!(scale >= 0.0f) || isinf(scale)) return USP_ERR_UNSUPPORTED;
  if (Lq >= (int64_t)1 << 31 || Lk >= (int64_t)1 << 31) return USP_ERR_UNSUPPORTED;
  if (state_bytes < attn_fwd_state_bytes(bs, Lq, hq, hs) || ((uintptr_t)state & 15)) return USP_ERR_WORKSPACE;
  usp_posdesc qd = {0, Lq, 0, 0}, kd = {0, Lk, 0, 0};
  if (causal) {
    if (!qpos || !kpos) return USP_ERR_NULL;
    if (!desc_ok(qpos, Lq) || !desc_ok(kpos, Lk)) return USP_ERR_SHAPE;
    qd = *qpos;
    kd = *kpos;
  }
  if (scale == 0.0f) scale = 1.0f / sqrtf((float)hs);
  const RingState rs = {(float*)state, first ? 1 : 0, last ? 1 : 0};
  return launch_block_attn_fwd(q, k, v, o, lse, bs, Lq, Lk, hq, hkv, hs, scale, causal ? 1 : 0, qd, kd, USP_BF16, o_dtype,
                               (hipStream_t)stream, &rs);
} catch (...) {
  return USP_ERR_LAUNCH;
}

namespace {
int ring_attn_fwd_impl(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                       const usp_posdesc* kpos_blocks, int n_blocks, void* o, float* lse, int bs, int64_t Lq,
                       int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc* qpos,
                       int in_dtype, int o_dtype, void* stream, bool v_transposed);
}  // namespace

extern "C" int usp_ring_attn_fwd(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                                 const usp_posdesc* kpos_blocks, int n_blocks, void* o, float* lse, int bs, int64_t Lq,
                                 int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc* qpos,
                                 int in_dtype, int o_dtype, void* stream) try {
  return ring_attn_fwd_impl(q, k_blocks, v_blocks, kpos_blocks, n_blocks, o, lse, bs, Lq, Lk, hq, hkv, hs, scale, causal,
                            qpos, in_dtype, o_dtype, stream, false);
} catch (...) {
  return USP_ERR_LAUNCH;
}

extern "C" int usp_ring_attn_fwd_vt(const void* q, const void* const* k_blocks, const void* const* vt_blocks,
                                    const usp_posdesc* kpos_blocks, int n_blocks, void* o, float* lse, int bs,
                                    int64_t Lq, int64_t Lk, int hq, int hkv, int hs, float scale, int causal,
                                    const usp_posdesc* qpos, void* stream) try {
  return ring_attn_fwd_impl(q, k_blocks, vt_blocks, kpos_blocks, n_blocks, o, lse, bs, Lq, Lk, hq, hkv, hs, scale, causal,
                            qpos, USP_BF16, USP_BF16, stream, true);
} catch (...) {
  return USP_ERR_LAUNCH;
}

namespace {
int ring_attn_fwd_impl(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                       const usp_posdesc* kpos_blocks, int n_blocks, void* o, float* lse, int bs, int64_t Lq,
                       int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc* qpos,
                       int in_dtype, int o_dtype, void* stream, bool v_transposed) {
  if (!q || !k_blocks || !v_blocks || !o || !lse) return USP_ERR_NULL;
  if (n_blocks < 1 || n_blocks > USP_MAX_RING_BLOCKS) return USP_ERR_UNSUPPORTED;
  if (bs < 1 || Lq < 1 || Lk < 1 || hq < 1 || hkv < 1) return USP_ERR_SHAPE;
  if (hq % hkv) return USP_ERR_DEGREE;
  if (hs != 64 && hs != 128) return USP_ERR_UNSUPPORTED;
  if (in_dtype != USP_BF16 || (o_dtype != USP_BF16 && o_dtype != USP_FP32)) return USP_ERR_DTYPE;
  if (!(scale >= 0.0f) || isinf(scale)) return USP_ERR_UNSUPPORTED;
  if (Lq >= (int64_t)1 << 31 || Lk >= (int64_t)1 << 31) return USP_ERR_UNSUPPORTED;
  usp_posdesc qd = {0, Lq, 0, 0};
  usp_posdesc kd[USP_MAX_RING_BLOCKS];
  if (causal && (!qpos || !kpos_blocks)) return USP_ERR_NULL;
  if (causal && !desc_ok(qpos, Lq)) return USP_ERR_SHAPE;
  if (causal) qd = *qpos;
  for (int j = 0; j < n_blocks; ++j) {
    if (!k_blocks[j] || !v_blocks[j]) return USP_ERR_NULL;
    kd[j] = usp_posdesc{0, Lk, 0, 0};
    if (causal) {
      if (!desc_ok(&kpos_blocks[j], Lk)) return USP_ERR_SHAPE;
      kd[j] = kpos_blocks[j];
    }
  }
  if (scale == 0.0f) scale = 1.0f / sqrtf((float)hs);
  if (v_transposed)
    for (int j = 0; j < n_blocks; ++j)
      if ((uintptr_t)v_blocks[j] & 15) return USP_ERR_UNSUPPORTED;
  return launch_ring_attn_fwd(q, k_blocks, v_blocks, kd, n_blocks, o, lse, bs, Lq, Lk, hq, hkv, hs, scale,
                              causal ? 1 : 0, qd, in_dtype, o_dtype, (hipStream_t)stream, nullptr, nullptr, v_transposed);
}
}  // namespace

extern "C" int usp_ring_attn_fwd_partials(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                                          const usp_posdesc* kpos_blocks, const int32_t* lk_blocks, int n_blocks,
                                          float* const* o_parts, float* const* lse_parts, int bs, int64_t Lq,
                                          int64_t Lk, int hq, int hkv, int hs, float scale, int causal,
                                          const usp_posdesc* qpos, void* stream) try {
  if (!q || !k_blocks || !v_blocks || !o_parts || !lse_parts) return USP_ERR_NULL;
  if (n_blocks < 1 || n_blocks > USP_MAX_RING_BLOCKS) return USP_ERR_UNSUPPORTED;
  if (bs < 1 || Lq < 1 || Lk < 1 || hq < 1 || hkv < 1) return USP_ERR_SHAPE;
  if (hq % hkv) return USP_ERR_DEGREE;
  if (hs != 64 && hs != 128) return USP_ERR_UNSUPPORTED;
  if (!(scale >= 0.0f) || isinf(scale)) return USP_ERR_UNSUPPORTED;
  if (Lq >= (int64_t)1 << 31 || Lk >= (int64_t)1 << 31) return USP_ERR_UNSUPPORTED;
  usp_posdesc qd = {0, Lq, 0, 0};
  usp_posdesc kd[USP_MAX_RING_BLOCKS];
  int lk[USP_MAX_RING_BLOCKS];
  if (causal && (!qpos || !kpos_blocks)) return USP_ERR_NULL;
  if (causal && !desc_ok(qpos, Lq)) return USP_ERR_SHAPE;
  if (causal) qd = *qpos;
  for (int j = 0; j < n_blocks; ++j) {
    if (!k_blocks[j] || !v_blocks[j] || !o_parts[j] || !lse_parts[j]) return USP_ERR_NULL;
    lk[j] = lk_blocks ? lk_blocks[j] : (int)Lk;
    if (lk[j] < 1 || lk[j] > Lk) return USP_ERR_SHAPE;
    kd[j] = usp_posdesc{0, lk[j], 0, 0};
    if (causal) {
      if (!desc_ok(&kpos_blocks[j], lk[j])) return USP_ERR_SHAPE;
      kd[j] = kpos_blocks[j];
    }
  }
  if (scale == 0.0f) scale = 1.0f / sqrtf((float)hs);
  return launch_attn_fwd_partials(q, k_blocks, v_blocks, kd, lk, n_blocks, o_parts, lse_parts, bs, Lq, Lk, hq, hkv, hs,
                                  scale, causal ? 1 : 0, qd, (hipStream_t)stream);
} catch (...) {
  return USP_ERR_LAUNCH;
}

extern "C" int usp_lse_merge(const void* const* o_parts, const float* const* lse_parts, int n_parts, void* o_out,
                             float* lse_out, int bs, int64_t Lq, int hq, int hs, int part_dtype, int out_dtype,
                             void* stream) {
  if (!o_parts || !lse_parts || !o_out || !lse_out) return USP_ERR_NULL;
  if (n_parts < 1 || n_parts > USP_MAX_MERGE_PARTS) return USP_ERR_UNSUPPORTED;
  for (int i = 0; i < n_parts; ++i)
    if (!o_parts[i] || !lse_parts[i]) return USP_ERR_NULL;
  if (bs < 1 || Lq < 1 || hq < 1 || hs < 1) return USP_ERR_SHAPE;
  if (hs % 8) return USP_ERR_UNSUPPORTED;
  if ((part_dtype != USP_BF16 && part_dtype != USP_FP32) || (out_dtype != USP_BF16 && out_dtype != USP_FP32))
    return USP_ERR_DTYPE;
  // An output may be the very buffer of a part only where the kernel is in-place safe: same element size (a thread
  // overwrites exactly the bytes it has read) and a row's threads inside one wavefront (hs / 4 divides 64), so that
  // the row's reads of the part's LSE precede the one store to it.  Any other overlap would read overwritten data.
  {
    const size_t rows = (size_t)bs * (size_t)Lq * hq;
    const size_t ob = rows * hs * dtype_size(out_dtype), pb = rows * hs * dtype_size(part_dtype), lb = rows * sizeof(float);
    const bool in_place_ok = part_dtype == out_dtype && (hs == 64 || hs == 128);
    for (int i = 0; i < n_parts; ++i) {
      if (overlap(o_out, ob, o_parts[i], pb) && !(in_place_ok && o_out == o_parts[i])) return USP_ERR_UNSUPPORTED;
      if (overlap(lse_out, lb, lse_parts[i], lb) && !(in_place_ok && lse_out == lse_parts[i])) return USP_ERR_UNSUPPORTED;
      if (overlap(o_out, ob, lse_parts[i], lb) || overlap(lse_out, lb, o_parts[i], pb)) return USP_ERR_UNSUPPORTED;
    }
  }
  return launch_lse_merge(o_parts, lse_parts, n_parts, o_out, lse_out, bs, Lq, hq, hs, part_dtype, out_dtype,
                          (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------------
// Algorithm 1 forward.  Workspace plan (all sizes rounded up to 256 B):
//   kv_head : K and V in head layout for every (ring row, Ulysses column in range): the ring loop of
//             a rank reads block s = (r - i) mod R of its own column u;
//   q_head, o_head : one rank's Q / O in head layout (reused rank after rank, stream-ordered); only on the
//             step-by-step path (the one-launch ring loop reads and writes the sequence-layout shards itself);
//   parts   : R partial O (fp32) + R partial LSE when R > 1.
// ---------------------------------------------------------------------------------------------
namespace {

inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

struct FwdPlan {
  size_t q_head, o_head, k_head, v_head, o_parts, lse_parts, total;
  size_t kv_block_bytes, v_block_bytes, part_o_bytes, part_lse_bytes;
  int n_cols;
  bool v_transposed;   // V blocks are staged in key-tile-transposed layout (the one-launch ring loop reads them so)
  // Ulysses degree 1: a K/V block in head layout IS its sequence-layout shard.  A batch of one: the shards of a ring row
  // are contiguous, and a block is they with the rank's heads inside longer rows.  K is then never staged; V only when it
  // is wanted in transposed tiles and re-tiling it costs less than the tiles save.
  bool k_in_place, v_in_place;
};

// Ulysses columns touched by ranks [rb, re): all U when the range spans more than one ring row.
void column_range(const usp_problem& p, int rb, int re, int* c0, int* c1) {
  const int U = p.ulysses;
  if (re - rb >= U || (rb / U) != ((re - 1) / U)) {
    *c0 = 0;
    *c1 = U;
  } else {
    *c0 = rb % U;
    *c1 = (re - 1) % U + 1;
  }
}

// The ring loop of a rank runs as one launch (state in registers, no partials, no merge) when the kernel family
// supports it: bf16 data and few enough blocks for the launch arguments.
bool ring_in_one_launch(const usp_problem& p) { return p.dtype == USP_BF16 && p.ring <= USP_MAX_RING_BLOCKS; }

// Key split of a rank's ring loop (launch_attn_fwd_partials): 0 = none (one work item per query tile, head and
// batch walks all blocks), else the number of pieces each K/V block is cut into, every piece of every block then
// being a work item of its own with a partial result of its own (1: the blocks themselves, for R > 1).  In the
// unsplit launch the item of the last query tile walks every key, which takes ratio = 256 / (items x 1/2 under
// a causal mask) times a CU's fair share of the whole launch.  Split from a ratio of 1.5: into two parts in all, three
// from a ratio of 3.5, four from 7 (the R blocks as they are when that is already as many or more); more parts cost
// more in partial results (fp32, written and merged) than they gain, and with one or two items per CU the finish time
// is a bin-packing matter (measured at L = 8192 and 16384: 2 and 3 pieces 1.4-1.8 x faster than none, 4 and more slower
// again; at L = 4096: 76 / 64 / 58 us with 2 / 3 / 4).  Pieces hold at least 1024 keys, and a launch takes no more parts in
// all than it takes blocks.  Host arithmetic only, with the chip's CU count as a constant (kPlanCUs): the workspace
// query must not need a GPU.
int key_splits(const usp_problem& p) {
  if (!ring_in_one_launch(p)) return 0;
  const int64_t Lq = p.L / p.ring;
  const int64_t items = ((Lq + 255) / 256) * (p.hc / p.ulysses) * p.bs;
  const double ratio = (double)kPlanCUs / ((double)items * (p.causal ? 0.5 : 1.0));
  if (ratio < 1.5) return 0;
  const int64_t parts_wanted = ratio >= 7.0 ? 4 : ratio >= 3.5 ? 3 : 2;
  int64_t s = (parts_wanted + p.ring - 1) / p.ring;
  s = std::min<int64_t>(s, Lq / 1024);
  s = std::min<int64_t>(s, USP_MAX_RING_BLOCKS / p.ring);
  s = std::max<int64_t>(s, 1);
  return s * p.ring > 1 ? (int)s : 0;
}

// Short of full grids (fewer than two work items per CU under a causal mask, the heaviest item longer than a CU's
// fair share) only the heaviest query tiles may be cut: the LAST `tiles` query tiles of the rank run as one item per
// piece of the keys (2 to 4 equal pieces of the one block when R = 1, else the R ring blocks), with fp32 partial results
// that are merged afterwards; the other tiles stay whole items of the same launch (launch_attn_fwd_partials with
// MixedLaunch).  How many tiles and pieces, if any, is decided by playing the launch through on the host: the kernel's
// own dealing (the first items given one per workgroup, the rest drawn in order by whoever is free), 8 us per item,
// 1.85 us per tile of 64 keys, 3 us each time a whole item moves on to another piece, and the merge of the cut rows at
// 5 TB/s + 10 us.  Host arithmetic only; the same for every Ulysses column of a ring row.
constexpr int kMaxHeavyPieces = USP_MAX_RING_BLOCKS;
struct HeavyPieces { int n; int64_t first[kMaxHeavyPieces], last[kMaxHeavyPieces]; int block[kMaxHeavyPieces]; };
struct HeavyChoice { int tiles, pieces; };   // tiles == 0: nothing is cut this way

// What a rank's launch runs: a list of items (listed_item()), heaviest first, over the pieces hp of the keys.  Piece j's
// partial result holds the rows from row0[j] on; the rows from merge_row0 on are merged.  No items: not planned this way.
struct ItemPlan {
  HeavyPieces hp;
  int64_t row0[kMaxHeavyPieces];
  int64_t merge_row0;
  std::vector<uint16_t> items;
};

// The pieces of a ring rank's keys, in the order its ring loop visits them: piece j = keys [first, last) of the block
// of ring step block[j].  R = 1: `pieces` equal parts of the one block (multiples of 64 keys); R > 1: the blocks.
HeavyPieces heavy_pieces(const usp_problem& p, int pieces) {
  HeavyPieces hp;
  const int64_t Lq = p.L / p.ring;
  if (p.ring == 1) {
    const int64_t piece = ((Lq + pieces - 1) / pieces + 63) / 64 * 64;
    hp.n = 0;
    for (int64_t a0 = 0; a0 < Lq; a0 += piece, ++hp.n) {
      hp.first[hp.n] = a0; hp.last[hp.n] = std::min(Lq, a0 + piece); hp.block[hp.n] = 0;
    }
  } else {
    hp.n = p.ring;
    for (int i = 0; i < p.ring; ++i) { hp.first[i] = 0; hp.last[i] = Lq; hp.block[i] = i; }
  }
  return hp;
}

// Positions of the keys [a, b) of a block whose positions are d.
usp_posdesc piece_of(const usp_posdesc& d, int64_t a, int64_t b) {
  if (a >= d.len0) return usp_posdesc{d.start1 + (a - d.len0), b - a, 0, 0};
  const int64_t n0 = std::min(b, d.len0) - a;
  return usp_posdesc{d.start0 + a, n0, d.start1, (b - a) - n0};
}

// A launch played through on the host: kPlanCUs workgroups, the one that is free first takes the next item, every item for
// `heads` heads and batch entries one behind the other.  As many workgroups as heads and workgroups have a common divisor
// always do the same, and one plays for all of them.
class PlayedLaunch {
 public:
  explicit PlayedLaunch(int heads) : alike_(std::gcd(heads, kPlanCUs)), workgroups_(kPlanCUs / alike_), copies_(heads / alike_) {}
  // an item of `us` for every head; false if one is not done before `limit`
  bool give(double us, double limit) {
    for (int c = 0; c < copies_; ++c) {
      const double done = give_one(us);
      end_ = std::max(end_, done);
      if (done >= limit) return false;
    }
    return true;
  }
  double end() const { return end_; }

 private:
  double give_one(double us) {
    if (n_ < workgroups_) {
      free_at_[n_++] = us;
      if (n_ == workgroups_) std::make_heap(free_at_, free_at_ + n_, std::greater<double>());
      return us;
    }
    const double done = free_at_[0] + us;
    int at = 0;   // the first one's new place in the heap
    for (int child; (child = 2 * at + 1) < n_; at = child) {
      if (child + 1 < n_ && free_at_[child + 1] < free_at_[child]) ++child;
      if (free_at_[child] >= done) break;
      free_at_[at] = free_at_[child];
    }
    free_at_[at] = done;
    return done;
  }
  int alike_, workgroups_, copies_, n_ = 0;
  double end_ = 0.0;
  double free_at_[kPlanCUs];
};

// What ring rank r cuts ({0, 0}: nothing, the launch is key_splits()' business): the room for partial results that the
// workspace has, and the cut itself where work_out_items() has none.  (Worked out once per problem: plans_of() below keeps
// the answers.)
HeavyChoice work_out_heavy_choice(const usp_problem& p, int r) {
  const HeavyChoice none = {0, 0};
  if (!ring_in_one_launch(p)) return none;
  const int64_t Lq = p.L / p.ring;
  usp_posdesc qd;
  ring_block_desc(p, r, &qd);
  const RowTiles rows(qd, Lq, p.causal);
  const int T = rows.n, n = (p.hc / p.ulysses) * p.bs;
  const int64_t items = (int64_t)T * n;
  if (items > 4 * kPlanCUs || Lq < 4096 || T < 8) return none;
  if (p.ring > 1 && items <= kPlanCUs) return none;   // short ring ranks: every tile per block, as key_splits() has it
  // Without a mask all items weigh the same and what is lost is the last, partly filled round (320 items on 256 CUs
  // take two rounds): the cut tiles' pieces then fill the first round and the whole items follow.
  if (!p.causal && items <= kPlanCUs) return none;
  const double kItem = 8.0, kTile = 1.85, kCross = 3.0;
  auto pos_of = [&](int64_t i) { return i < qd.len0 ? qd.start0 + i : qd.start1 + (i - qd.len0); };
  // 64-key tiles of piece j that query tile i walks: under kpos <= qpos the visible keys of each run are a prefix of it
  std::vector<double> tiles;
  auto look = [&](const HeavyPieces& hp) {
    tiles.resize((size_t)T * hp.n);
    for (int j = 0; j < hp.n; ++j) {
      usp_posdesc kd;
      ring_block_desc(p, ((r - hp.block[j]) % p.ring + p.ring) % p.ring, &kd);
      const usp_posdesc pd = piece_of(kd, hp.first[j], hp.last[j]);
      for (int i = 0; i < T; ++i) {
        const int64_t a = rows.begin(i), b = rows.end(i);
        int64_t qmax = std::max(pos_of(a), pos_of(b - 1));
        if (a < qd.len0 && b > qd.len0) qmax = std::max({qmax, pos_of(qd.len0 - 1), pos_of(qd.len0)});
        const int64_t c0 = p.causal ? std::clamp<int64_t>(qmax - pd.start0 + 1, 0, pd.len0) : pd.len0;
        const int64_t c1 = p.causal ? std::clamp<int64_t>(qmax - pd.start1 + 1, 0, pd.len1) : pd.len1;
        tiles[(size_t)i * hp.n + j] = (double)((c0 + 63) / 64 + (c1 + 63) / 64);
      }
    }
  };
  // time of the launch with the last k query tiles cut into the pieces hp, looked at before (k = T: every tile, k = 0: none);
  // `limit` if it is that or more
  auto launch_time = [&](const HeavyPieces& hp, int k, double limit) {
    auto whole = [&](int t) {
      double sum = 0.0;
      int walked = 0;
      for (int j = 0; j < hp.n; ++j) {
        sum += tiles[(size_t)(T - 1 - t) * hp.n + j];
        walked += tiles[(size_t)(T - 1 - t) * hp.n + j] > 0.0;
      }
      // (the one-launch ring loop pays the change of block too, so it is charged whether or not anything is cut)
      const double cross = (p.ring > 1 || k > 0) ? kCross * std::max(0, walked - 1) : 0.0;
      return kItem + kTile * sum + cross;
    };
    const double cut_rows = (double)(Lq - rows.begin(T - k)) * n;
    const double merge_us = k > 0 ? 10.0 + cut_rows * p.hs * (hp.n * 2.0 * 4.0 + 2.0) / 5.0e6 : 0.0;   // the fp32 partials written and read, bf16 out
    double work = 0.0;   // less than a fair share of it is not possible
    for (int t = 0; t < k; ++t)
      for (int j = 0; j < hp.n; ++j) work += kItem + kTile * tiles[(size_t)(T - 1 - t) * hp.n + j];
    for (int t = k; t < T; ++t) work += whole(t);
    if (work * n / kPlanCUs * (1.0 - 1e-9) + merge_us >= limit) return limit;
    PlayedLaunch launch(n);
    for (int t = 0; t < k; ++t)
      for (int j = 0; j < hp.n; ++j)
        if (!launch.give(kItem + kTile * tiles[(size_t)(T - 1 - t) * hp.n + j], limit - merge_us)) return limit;
    for (int t = k; t < T; ++t)
      if (!launch.give(whole(t), limit - merge_us)) return limit;
    return launch.end() + merge_us;
  };
  // what the launch costs as key_splits() has it: whole, or every tile in so many pieces per block
  const int splits = key_splits(p);
  const HeavyPieces as_is = heavy_pieces(p, splits > 0 ? splits : 2);
  look(as_is);
  const double as_is_us = launch_time(as_is, splits > 0 ? T : 0, 1e30);
  // A cut has to pay for itself: 3 % by this model when the pieces are parts of one block and the launch was whole,
  // where the model's choice was the measured optimum at every length tried; 8 % when they are ring blocks of unequal
  // visible parts, where it promises 5 % more than is measured (the uncut launch's long tail runs on few CUs at a
  // higher clock); 5 % against a launch that already cuts every tile.
  const double need = p.ring > 1 ? 0.92 : splits > 0 ? 0.95 : 0.97;
  HeavyChoice best = none;
  double best_us = as_is_us;
  for (int pieces = 2; pieces <= (p.ring == 1 ? 4 : 2); ++pieces) {   // (R > 1: the blocks, one pass)
    if (p.ring == 1 && Lq / pieces < 1024) break;
    const HeavyPieces hp = heavy_pieces(p, pieces);
    look(hp);
    for (int part = 1; part < 32; ++part) {   // k in steps of T / 32
      const int k = std::max(1, T * part / 32);
      if (part > 1 && k == std::max(1, T * (part - 1) / 32)) continue;
      const double us = launch_time(hp, k, best_us);
      if (us < best_us) { best = HeavyChoice{k, hp.n}; best_us = us; }
    }
  }
  if (best_us >= need * as_is_us) return none;
  return best;
}

// The launch of ring rank r within the room that the plan has for partial results (that of choice, or of key_splits()): which
// tiles are cut, into which pieces, by playing the launch through for a number of cuts.  Items are dealt heaviest first, a
// tile's pieces that it sees nothing of are none, and a partial result holds only the rows that see its piece, so that the
// room for three whole ones is room for four or five.  Measured against equal pieces for the last tiles, every pair of tile and
// piece an item (an empty one took 9 us to write zeros), whole usp_attn_fwd of one rank, us: 32/8 heads, U 8: L = 6144 70.9 ->
// 65.9, 8192 97.2 -> 90.6, 10240 147 -> 127, 12288 181 -> 168, 16384 275 -> 274, 20480 428 -> 405, 24576 594 -> 569; U 4 x R 2,
// L = 16384, rank 0 292 -> 278, 7 337 -> 287; U 8 x R 2, L = 40960, rank 0 1000 -> 828, 8 820 -> 826; R 8, L = 8192, rank 0 131 -> 118,
// 7 133 -> 132; head size 64, U 8, L = 12288 119 -> 105.  500 random ranks 1.09 times as fast, three of them slower by more than
// 2 %; known to be slower: rings of four and eight contiguous blocks whose equal items just do not fit the CUs once more (32/1 heads,
// R 4, L = 3776 82 -> 84; R 8, 4448 82 -> 86 to 91), and without a mask 18 tiles of 16 heads (U 2, L = 4444 180 -> 185).  The answer is
// within the room that callers have been told.
constexpr int kMaxMergeRowParts = 8;   // (launch_lse_merge)
ItemPlan work_out_items(const usp_problem& p, int r, const HeavyChoice& choice) {
  ItemPlan best;
  best.hp.n = 0;
  best.merge_row0 = 0;
  const int64_t Lq = p.L / p.ring;
  const int room = std::max(key_splits(p) * p.ring, choice.tiles > 0 ? choice.pieces : 0);   // partial results of all rows
  if (room == 0 || !ring_in_one_launch(p)) return best;
  usp_posdesc qd;
  ring_block_desc(p, r, &qd);
  const RowTiles rows(qd, Lq, p.causal);
  const int T = rows.n, n = (p.hc / p.ulysses) * p.bs;
  if (T > kMaxListedItems || (int64_t)T * n > 4 * kPlanCUs) return best;
  // us of an item besides its tiles, of a tile of 64 keys, of a whole item's step to the next piece; read off time stamps (at head
  // size 64 before the second product ran a tile behind: its tile is 1.06 to 1.1 since; the other estimates of that head size, of
  // the choice above and of the launches that split keys over waves, are of then too)
  const double kItem = 9.0, kTile = p.hs == 128 ? 1.78 : 1.15, kCross = 3.0;
  auto pos_of = [&](int64_t i) { return i < qd.len0 ? qd.start0 + i : qd.start1 + (i - qd.len0); };
  std::vector<int64_t> qmax(T);
  for (int i = 0; i < T; ++i) {
    const int64_t a = rows.begin(i), b = rows.end(i);
    qmax[i] = std::max(pos_of(a), pos_of(b - 1));
    if (a < qd.len0 && b > qd.len0) qmax[i] = std::max({qmax[i], pos_of(qd.len0 - 1), pos_of(qd.len0)});
  }
  struct Item { double us; uint16_t entry; };
  std::vector<Item> list;
  std::vector<int> sees;   // [tile][piece]: tiles of 64 keys that query tile i walks in piece j
  std::vector<double> whole(T), cut(T), longest(T + 1);   // us of tile i's one item, of its items per piece, the longest item from i on if cut
  std::vector<double> whole_before(T + 1), cut_from(T + 1);
  int first_seeing[kMaxHeavyPieces];   // the query tile from which on the piece is seen
  double best_us = 1e30;
  auto look = [&](const HeavyPieces& hp) {
    sees.resize((size_t)T * hp.n);
    std::fill(whole.begin(), whole.end(), 0.0);
    std::fill(cut.begin(), cut.end(), 0.0);
    std::fill(longest.begin(), longest.end(), 0.0);
    for (int j = 0; j < hp.n; ++j) {
      usp_posdesc kd;
      ring_block_desc(p, ((r - hp.block[j]) % p.ring + p.ring) % p.ring, &kd);
      const usp_posdesc pd = piece_of(kd, hp.first[j], hp.last[j]);
      first_seeing[j] = T;
      for (int i = T - 1; i >= 0; --i) {   // (rows stand in ascending order: what sees a piece is a run of tiles up to the last)
        const int64_t c0 = p.causal ? std::clamp<int64_t>(qmax[i] - pd.start0 + 1, 0, pd.len0) : pd.len0;
        const int64_t c1 = p.causal ? std::clamp<int64_t>(qmax[i] - pd.start1 + 1, 0, pd.len1) : pd.len1;
        const int n_tiles = (int)((c0 + 63) / 64 + (c1 + 63) / 64);
        sees[(size_t)i * hp.n + j] = n_tiles;
        if (n_tiles == 0) continue;
        first_seeing[j] = i;
        whole[i] += kTile * n_tiles + kCross;
        cut[i] += kItem + kTile * n_tiles;
        longest[i] = std::max(longest[i], kItem + kTile * n_tiles);
      }
    }
    whole_before[0] = cut_from[T] = 0.0;
    for (int i = 0; i < T; ++i) {
      whole[i] = kItem + std::max(0.0, whole[i] - kCross);
      whole_before[i + 1] = whole_before[i] + whole[i];
    }
    for (int i = T - 1; i >= 0; --i) {
      cut_from[i] = cut_from[i + 1] + cut[i];
      longest[i] = std::max(longest[i], longest[i + 1]);
    }
  };
  // the last k tiles cut into hp (looked at before)
  auto consider = [&](const HeavyPieces& hp, int k) {
    if (k < 1 || k > T) return;
    int64_t row0[kMaxHeavyPieces], held = 0;
    for (int j = 0; j < hp.n; ++j) {
      const int first = std::max(T - k, first_seeing[j]);
      row0[j] = first < T ? rows.begin(first) : Lq;
      held += Lq - row0[j];
    }
    const int64_t cut_row0 = rows.begin(T - k);
    if (row0[0] > cut_row0 || held > room * Lq) return;
    const double merge_us = 10.0 + ((double)held * 8.0 + (double)(Lq - cut_row0) * 2.0) * n * p.hs / 5.0e6;
    // no sooner than a fair share, and than the longest item
    if ((whole_before[T - k] + cut_from[T - k]) * n / kPlanCUs * (1.0 - 1e-9) + merge_us >= best_us || longest[T - k] + merge_us >= best_us ||
        (k < T && whole[T - k - 1] + merge_us >= best_us))
      return;
    list.clear();
    for (int i = 0; i < T - k; ++i) list.push_back({whole[i], listed_item(i, kListedWhole)});
    for (int i = T - k; i < T; ++i)
      for (int j = 0; j < hp.n; ++j)
        if (const int n_tiles = sees[(size_t)i * hp.n + j]) list.push_back({kItem + kTile * n_tiles, listed_item(i, j)});
    if ((int)list.size() > kMaxListedItems) return;
    std::stable_sort(list.begin(), list.end(), [](const Item& a, const Item& b) { return a.us > b.us; });
    // of the first m kPlanCUs + 1 items some workgroup has m + 1, none shorter than the last of these
    for (size_t m = 1; m * kPlanCUs < list.size() * n; ++m)
      if ((m + 1) * list[m * kPlanCUs / n].us + merge_us >= best_us) return;
    PlayedLaunch launch(n);
    for (const Item& it : list)
      if (!launch.give(it.us, best_us - merge_us)) return;
    if (launch.end() + merge_us >= best_us) return;
    best_us = launch.end() + merge_us;
    best.hp = hp;
    std::copy(row0, row0 + hp.n, best.row0);
    best.merge_row0 = cut_row0;
    best.items.clear();
    for (const Item& it : list) best.items.push_back(it.entry);
  };
  auto cut_last = [&](const HeavyPieces& hp) {
    look(hp);
    for (int part = 1; part <= 32; ++part) {
      const int k = std::max(1, T * part / 32);
      if (part == 1 || k != std::max(1, T * (part - 1) / 32)) consider(hp, k);
    }
  };
  if (p.ring > 1) {   // the blocks, whole or in as many pieces as key_splits() has them
    for (int m = 1; m * p.ring <= kMaxMergeRowParts && m <= std::max(1, key_splits(p)); ++m) {
      HeavyPieces hp;
      hp.n = 0;
      const int64_t piece = ((Lq + m - 1) / m + 63) / 64 * 64;
      for (int i = 0; i < p.ring; ++i)
        for (int64_t a = 0; a < Lq; a += piece, ++hp.n) {
          hp.first[hp.n] = a; hp.last[hp.n] = std::min(Lq, a + piece); hp.block[hp.n] = i;
        }
      cut_last(hp);
    }
    return best;
  }
  // Without a mask all items are as long, and what is left of a last round is dealt out in pieces: in eight it ends sooner than in
  // four (70 tiles of four heads are 256 items and 24 more, which as 96 pieces kept 96 CUs for a quarter of an item, as 192 pieces
  // 192 of them for an eighth).  us, up to four pieces -> up to eight: U 8: L = 17776 612 -> 579 (head size 64 384 -> 363), 16704
  // 563 -> 521, 25728 1209 -> 1195; U 4, L = 9000 332 -> 312; U 2, head size 64, 5216 146 -> 141; U 1, 16 heads, 4368 175 -> 167; of 24
  // lengths the others as before.  With a mask the lengths below are tried instead.
  for (int pieces = p.causal ? 4 : kMaxMergeRowParts; pieces >= 2; --pieces) cut_last(heavy_pieces(p, pieces));
  if (p.causal) {
    // pieces of so many keys that every item is about as long; tiles that see no more than one piece are whole
    const int tiles = (int)((Lq + 63) / 64);
    const int shortest = std::max(4, (tiles + kMaxMergeRowParts - 1) / kMaxMergeRowParts);
    for (int step = 0, q = tiles - 1; q >= shortest && step < 64; ++step, q -= std::max(1, tiles / 64)) {
      HeavyPieces hp;
      hp.n = 0;
      for (int64_t a = 0; a < Lq; a += 64 * q, ++hp.n) {
        hp.first[hp.n] = a; hp.last[hp.n] = std::min(Lq, a + 64 * q); hp.block[hp.n] = 0;
      }
      look(hp);
      int k = 0;
      while (k < T && hp.n > 1 && sees[(size_t)(T - 1 - k) * hp.n + 1] > 0) ++k;
      consider(hp, k);
    }
  }
  return best;
}

// (the scale plays no part in how a problem is cut)
bool same_problem(const usp_problem& a, const usp_problem& b) {
  return a.bs == b.bs && a.L == b.L && a.hc == b.hc && a.hk == b.hk && a.hs == b.hs && a.ulysses == b.ulysses &&
         a.ring == b.ring && a.causal == b.causal && a.split == b.split && a.dtype == b.dtype;
}

// Playing launches through takes the host 10 to 400 us per ring rank (L = 8192, U 8, 25 us for the choice and 80 for the items;
// 16384, U 4 x R 2, 28 for the items; 24576, U 8, 100 and 380; no mask, 17776, 120 and 330): the answers for the last problems
// asked about are kept.  Every ring rank's choice is worked out at the first question about the problem, for the workspace
// depends on all; a ring rank's items when it is first launched by them, or, where it is the only one, asked about.  Nobody waits for another problem's answers.
struct Plans {
  usp_problem p;
  std::vector<HeavyChoice> choices;
  std::mutex mu;
  std::vector<std::unique_ptr<const ItemPlan>> items;
  const ItemPlan& items_of(int r) {
    std::lock_guard<std::mutex> lock(mu);
    if (!items[r]) items[r] = std::make_unique<const ItemPlan>(work_out_items(p, r, choices[r]));
    return *items[r];
  }
};
std::shared_ptr<Plans> plans_of(const usp_problem& p) {
  static std::mutex mu;
  static std::vector<std::shared_ptr<Plans>> seen;   // the last asked about is last
  auto find = [&]() -> std::shared_ptr<Plans> {
    for (auto it = seen.rbegin(); it != seen.rend(); ++it)
      if (same_problem((*it)->p, p)) {
        std::rotate(it.base() - 1, it.base(), seen.end());
        return seen.back();
      }
    return nullptr;
  };
  {
    std::lock_guard<std::mutex> lock(mu);
    if (auto known = find()) return known;
  }
  auto plans = std::make_shared<Plans>();
  plans->p = p;
  for (int r = 0; r < p.ring; ++r) plans->choices.push_back(work_out_heavy_choice(p, r));
  plans->items.resize(p.ring);
  std::lock_guard<std::mutex> lock(mu);
  if (auto known = find()) return known;
  if (seen.size() >= 64) seen.erase(seen.begin());
  seen.push_back(plans);
  return plans;
}

// The most pieces any ring rank of the problem cuts its heaviest tiles into (0: no rank does): the workspace holds as
// many partial results.
int heavy_max_pieces(const usp_problem& p) {
  if (!ring_in_one_launch(p)) return 0;
  int m = 0;
  for (const HeavyChoice& c : plans_of(p)->choices)
    if (c.tiles > 0) m = std::max(m, c.pieces);
  return m;
}

// Short sequences: whether all ranks of a range go through the one launch of wave_split_attn_fwd.hip instead of two to
// four launches per rank, one rank after the other.  Those take at least 30 us (25 at head size 64) per rank and run at
// 1.15 (0.8) PFLOP/s beyond that, the one launch as wave_split_us() says.  Measured, per-rank launches against the one, us:
// 32/8 heads, U 8, one rank: L = 1024 37 / 11, 2048 34 / 18, 3072 37 / 24, 4096 43 / 37, 5120 54 / 59, 6144 68 / 79; without a mask
// L = 3072 45 / 45, 4096 57 / 64; batch of two L = 2048 42 / 23, 4096 71 / 73; U 1 (32 heads): L = 1024 39 / 31, 1536 52 / 53; head
// size 64, U 8: L = 4096 34 / 23, 6144 47 / 43, 8192 65 / 70, without a mask L = 4096 41 / 36, 6144 67 / 74; all four ranks of 8/4
// heads, U 2 x R 2: L = 1024 116 / 12, 4096 176 / 73.  (Two near the line that it has on the other side: batch of two, L = 3072
// 53 / 47; head size 64, U 1, L = 2048 52 / 43.)
bool short_in_one_launch(const usp_problem& p, int n_ranks) {
  const int64_t Lq = p.L / p.ring;
  const int heads = p.bs * (p.hc / p.ulysses);
  const double flop = 4.0 * p.hs * heads * (double)Lq * (double)p.L * (p.causal ? 0.5 : 1.0);   // of one rank
  const double by_rank = p.hs == 128 ? 30.0 + flop / 1.15e9 : 25.0 + flop / 0.8e9;
  return wave_split_us(Lq, heads * n_ranks, p.hs, flop * n_ranks) < by_rank * n_ranks;
}

// allow_heavy = false: as if no rank cut its heaviest tiles (the entry point without a workspace of its own falls back
// to that when the partials would not fit its array).  may_read_in_place = false: K or V does not lie on 16 bytes, as the
// kernels' reads of whole chunks want them, or the results go over them; the staged copies are neither.  (The sizes are
// the same.)
FwdPlan plan_fwd(const usp_problem& p, int n_cols, bool allow_heavy = true, bool may_read_in_place = true) {
  FwdPlan f;
  const size_t es = dtype_size(p.dtype);
  const size_t Lq = p.L / p.ring, hq = p.hc / p.ulysses, hkv = p.hk / p.ulysses;
  const size_t qb = up256((size_t)p.bs * Lq * hq * p.hs * es);
  f.kv_block_bytes = (size_t)p.bs * Lq * hkv * p.hs * es;   // exact: blocks are packed back to back (multiple of 128 B)
  f.part_o_bytes = up256((size_t)p.bs * Lq * hq * p.hs * sizeof(float));
  f.part_lse_bytes = up256((size_t)p.bs * Lq * hq * sizeof(float));
  f.n_cols = n_cols;
  size_t off = 0;
  // the one-launch ring loop reads Q from and writes O to the sequence-layout shards: no head-layout copies of them
  const size_t qo = ring_in_one_launch(p) ? 0 : qb;
  f.q_head = off; off += qo;
  f.o_head = off; off += qo;
  const int heavy = allow_heavy ? heavy_max_pieces(p) : 0;
  const int splits = key_splits(p);
  // The one-launch ring loop and the launch that cuts only the heaviest tiles (not the launch that cuts every tile,
  // whose fp32 instance reads V rows) take V in key-tile-transposed layout: tiles of 64 keys, the last one padded.
  // With Ulysses degree 1 the all-to-all of Algorithm 1 is the identity: block s in head layout, [bs][L/R][hk][hs], is
  // shard s as it stands, and the kernels read K where it is.  V too, as rows, unless re-tiling it (the only copy
  // left: all R blocks read and written at about 5 TB/s, one launch of about 6 us) costs less than the transposed
  // tiles save (1.3 % of the attention time, taken as visible pairs x 4 hs flop at 1.1 PFLOP/s).  Measured, one
  // ring-only rank of L = 32768, ring 8: 8 KV heads 1.014 -> 0.970 ms with both in place (0.987 estimated with V
  // re-tiled); one KV head 0.954 -> 0.960 ms with both in place, hence V re-tiled there.
  f.k_in_place = p.ulysses == 1;
  f.v_transposed = ring_in_one_launch(p) && splits == 0;
  auto retiling_pays = [&]() {
    const double pairs = (double)p.bs * hq * (double)Lq * (double)p.L * (p.causal ? 0.5 : 1.0);
    const double attention_us = pairs * 4.0 * p.hs / 1.1e9;
    const double retile_us = 2.0 * (double)p.bs * p.L * hkv * p.hs * es / 5e6 + 6.0;
    return retile_us <= 0.013 * attention_us;
  };
  if (f.k_in_place && f.v_transposed) f.v_transposed = retiling_pays();
  f.v_block_bytes = f.v_transposed ? vt_block_bytes(p.bs, (int64_t)Lq, (int)hkv, p.hs) : f.kv_block_bytes;
  f.k_head = off; off += f.k_in_place ? 0 : up256(f.kv_block_bytes * p.ring * n_cols);
  f.v_head = off; off += f.k_in_place && !f.v_transposed ? 0 : up256(f.v_block_bytes * p.ring * n_cols);
  // A batch of one is read in place at every Ulysses degree (the room for its staged copies stays in the plan: callers
  // have been told the size).  Measured, L = 8192, one of eight Ulysses ranks: 96.3 us staged, 92.8 in place; L = 32768 no
  // difference (924, 921).
  if (p.bs == 1 && may_read_in_place && !f.k_in_place && ring_in_one_launch(p)) {
    f.k_in_place = true;
    f.v_transposed = f.v_transposed && retiling_pays();
  }
  f.v_in_place = f.k_in_place && !f.v_transposed;
  size_t parts = splits > 0 ? (size_t)splits * p.ring : (p.ring > 1 && !ring_in_one_launch(p)) ? p.ring : 0;
  parts = std::max<size_t>(parts, (size_t)heavy);
  f.o_parts = off; off += f.part_o_bytes * parts;
  f.lse_parts = off; off += f.part_lse_bytes * parts;
  f.total = off;
  return f;
}

}  // namespace

namespace {

// V of every (ring row, Ulysses column in [c0, c1)) in key-tile-transposed layout, packed by slot r * n_cols + (u - c0).
int stage_vt_blocks(const usp_problem& p, const void* v, char* v_head, size_t block_bytes, int c0, int c1, hipStream_t stream) {
  const int U = p.ulysses, R = p.ring, n_cols = c1 - c0;
  if (n_cols == U) return launch_layout_a2a_vt(p, p.hk, v, v_head, 0, U * R, -1, stream);
  if (n_cols == 1) return launch_layout_a2a_vt(p, p.hk, v, v_head, c0, U * R, -1, stream, U);
  int st = USP_OK;
  for (int r = 0; r < R && st == USP_OK; ++r)
    st = launch_layout_a2a_vt(p, p.hk, v, v_head + (size_t)r * n_cols * block_bytes, r * U + c0, r * U + c1, -1, stream);
  return st;
}

// K and V of every (ring row, Ulysses column in [c0, c1)) to head layout, packed by slot r * n_cols + (u - c0).
int stage_kv_blocks(const usp_problem& p, const void* k, const void* v, char* k_head, char* v_head, size_t block_bytes,
                    int c0, int c1, hipStream_t stream, size_t vt_block_bytes_ = 0) {
  const int U = p.ulysses, R = p.ring, n_cols = c1 - c0;
  if (vt_block_bytes_) {
    // K as rows, V in key-tile-transposed layout: one launch each, same ranks and slots
    int st = USP_OK;
    const void* ksrc[1] = {k};
    void* kdst[1] = {k_head};
    if (n_cols == U) {
      st = launch_layout_a2a_multi(p, p.hk, USP_SEQ_TO_HEAD, 1, ksrc, kdst, 0, U * R, -1, stream);
    } else if (n_cols == 1) {
      st = launch_layout_a2a_multi(p, p.hk, USP_SEQ_TO_HEAD, 1, ksrc, kdst, c0, U * R, -1, stream, U);
    } else {
      for (int r = 0; r < R && st == USP_OK; ++r) {
        kdst[0] = k_head + (size_t)r * n_cols * block_bytes;
        st = launch_layout_a2a_multi(p, p.hk, USP_SEQ_TO_HEAD, 1, ksrc, kdst, r * U + c0, r * U + c1, -1, stream);
      }
    }
    return st == USP_OK ? stage_vt_blocks(p, v, v_head, vt_block_bytes_, c0, c1, stream) : st;
  }
  // K and V have one geometry: both go through the same launches
  const void* src[2] = {k, v};
  int st = USP_OK;
  if (n_cols == U) {
    void* dst[2] = {k_head, v_head};
    st = launch_layout_a2a_multi(p, p.hk, USP_SEQ_TO_HEAD, 2, src, dst, 0, U * R, -1, stream);
  } else if (n_cols == 1) {
    void* dst[2] = {k_head, v_head};
    st = launch_layout_a2a_multi(p, p.hk, USP_SEQ_TO_HEAD, 2, src, dst, c0, U * R, -1, stream, U);
  } else {
    for (int r = 0; r < R && st == USP_OK; ++r) {
      void* dst[2] = {k_head + (size_t)r * n_cols * block_bytes, v_head + (size_t)r * n_cols * block_bytes};
      st = launch_layout_a2a_multi(p, p.hk, USP_SEQ_TO_HEAD, 2, src, dst, r * U + c0, r * U + c1, -1, stream);
    }
  }
  return st;
}

}  // namespace

extern "C" size_t usp_attn_fwd_workspace_bytes(const usp_problem* p, int n_ranks) try {
  if (usp_validate(p) != USP_OK || n_ranks < 1) return 0;
  // one rank touches one Ulysses column; a wider range may straddle ring rows, so size for all U
  const int cols = n_ranks == 1 ? 1 : p->ulysses;
  const size_t bytes = plan_fwd(*p, cols).total;
  // (one ring rank: its items are the ones that will be launched, so they are worked out here and not in the first call)
  if (p->ring == 1 && ring_in_one_launch(*p) && !short_in_one_launch(*p, n_ranks)) plans_of(*p)->items_of(0);
  return bytes;
} catch (...) {
  return 0;
}

namespace {
int attn_fwd_impl(const usp_problem* p, const void* q, const void* k, const void* v, void* o, float* lse,
                  int rank_begin, int rank_end, void* workspace, size_t workspace_bytes, void* stream_,
                  bool allow_heavy = true) {
  int st = usp_validate(p);
  if (st != USP_OK) return st;
  if (!q || !k || !v || !o || !lse) return USP_ERR_NULL;
  const int U = p->ulysses, R = p->ring, N = U * R;
  if (rank_begin < 0 || rank_end > N || rank_begin >= rank_end) return USP_ERR_UNSUPPORTED;
  int c0, c1;
  column_range(*p, rank_begin, rank_end, &c0, &c1);
  const bool aligned = (((uintptr_t)k | (uintptr_t)v) & 15) == 0;
  const size_t es = dtype_size(p->dtype);
  const int64_t Lq = p->L / R;
  const int hq = p->hc / U, hkv = p->hk / U;
  // Results may only be written while inputs are still read if they share no memory (O over Q itself apart: whoever writes
  // rows of O has read these rows of Q, and nobody else reads them).
  bool kv_apart = true, q_apart = true;
  {
    const size_t ring_row = (size_t)p->bs * Lq * p->hc * p->hs * es, kv_all = (size_t)p->bs * p->L * p->hk * p->hs * es;
    const size_t lse_rank_bytes = (size_t)p->bs * hq * Lq * sizeof(float);
    const size_t first = rank_begin / U * ring_row, qo_bytes = ((rank_end - 1) / U + 1) * ring_row - first;
    const char *o_out = (const char*)o + first, *q_in = (const char*)q + first;
    const char* lse_out = (const char*)lse + rank_begin * lse_rank_bytes;
    const size_t lse_bytes = (rank_end - rank_begin) * lse_rank_bytes;
    for (const void* in : {k, v})
      if (overlap(in, kv_all, o_out, qo_bytes) || overlap(in, kv_all, lse_out, lse_bytes)) kv_apart = false;
    if ((o != q && overlap(q_in, qo_bytes, o_out, qo_bytes)) || overlap(q_in, qo_bytes, lse_out, lse_bytes)) q_apart = false;
  }
  const FwdPlan f = plan_fwd(*p, c1 - c0, allow_heavy, aligned && kv_apart);
  // (a plan that needs no workspace at all, as a ring-only problem in one launch, takes any pointer, null included)
  if (f.total > 0 && (!workspace || workspace_bytes < f.total || ((uintptr_t)workspace & 255))) return USP_ERR_WORKSPACE;
  hipStream_t stream = (hipStream_t)stream_;
  char* ws = (char*)workspace;
  const float scale = p->scale == 0.0f ? 1.0f / sqrtf((float)p->hs) : p->scale;

  // fp32 data, and short sequences: all ranks of the range in one launch that reads and writes the shards themselves
  // (results over inputs: step by step, from staged copies)
  if (p->dtype == USP_FP32 && R > USP_MAX_MERGE_PARTS) return USP_ERR_UNSUPPORTED;
  if (kv_apart && q_apart &&
      (p->dtype == USP_FP32 || (aligned && R <= USP_MAX_MERGE_PARTS && short_in_one_launch(*p, rank_end - rank_begin))))
    return launch_wave_split_usp_fwd(*p, q, k, v, o, lse, rank_begin, rank_end, scale, stream);

  // Steps 3-4 of Algorithm 1 for every K/V block the ranks in range will visit.  The workspace slot of
  // block (r, u) is r * n_cols + (u - c0): with all U columns that is the rank order (one launch per
  // tensor); with one column the ranks r * U + u are a stride-U sequence (again one launch per tensor).
  if (!f.k_in_place) {
    st = stage_kv_blocks(*p, k, v, ws + f.k_head, ws + f.v_head, f.kv_block_bytes, c0, c1, stream,
                         f.v_transposed ? f.v_block_bytes : 0);
    if (st != USP_OK) return st;
  } else if (!f.v_in_place) {
    st = stage_vt_blocks(*p, v, ws + f.v_head, f.v_block_bytes, c0, c1, stream);
    if (st != USP_OK) return st;
  }

  // K and V of ring row s for Ulysses rank u: in place, the row's shards from the rank's first KV head on (rows of hk
  // heads), else the workspace slot (rows of hkv heads)
  const int kv_pitch = f.k_in_place ? p->hk : hkv;
  auto kv_block = [&](bool in_place, const void* t, size_t region, size_t block_bytes, int s, int u) -> const char* {
    return in_place ? (const char*)t + ((size_t)s * p->bs * Lq * p->hk + (size_t)u * hkv) * p->hs * es
                    : ws + region + ((size_t)s * (c1 - c0) + (u - c0)) * block_bytes;
  };
  auto k_block = [&](int s, int u) { return kv_block(f.k_in_place, k, f.k_head, f.kv_block_bytes, s, u); };
  auto v_block = [&](int s, int u) { return kv_block(f.v_in_place, v, f.v_head, f.v_block_bytes, s, u); };

  const auto plans = allow_heavy && ring_in_one_launch(*p) ? plans_of(*p) : nullptr;
  for (int rank = rank_begin; rank < rank_end; ++rank) {
    const int r = rank / U, u = rank % U;
    // Step 2: Q of this rank to head layout (the one-launch ring loop reads the shards itself).
    if (!ring_in_one_launch(*p)) {
      st = launch_layout_a2a(*p, p->hc, USP_SEQ_TO_HEAD, q, ws + f.q_head, rank, rank + 1, rank, stream);
      if (st != USP_OK) return st;
    }
    usp_posdesc qd;
    usp_local_positions(p, r, u, nullptr, &qd);
    float* lse_rank = lse + (size_t)rank * p->bs * hq * Lq;
    // Step 5: the ring loop.  Step i visits block s = (r - i) mod R.
    if (ring_in_one_launch(*p)) {
      const void* kb[USP_MAX_RING_BLOCKS];
      const void* vb[USP_MAX_RING_BLOCKS];
      usp_posdesc kds[USP_MAX_RING_BLOCKS];
      for (int i = 0; i < R; ++i) {
        const int s = ((r - i) % R + R) % R;
        usp_local_positions(p, s, u, nullptr, &kds[i]);
        kb[i] = k_block(s, u);
        vb[i] = v_block(s, u);
      }
      // Steps 2 and 6 for Q and O ride on the kernel's own accesses: it reads each Q row once and writes each O
      // row once, so it does that straight from / to the sequence-layout shards of the Ulysses group.
      const SeqLayoutIO seq = {(int)(p->L / N), p->hc, u * hq, kv_pitch};
      const size_t group_off = (size_t)r * U * p->bs * (p->L / N) * p->hc * p->hs * es;
      const ItemPlan* const list = plans ? &plans->items_of(r) : nullptr;
      const HeavyChoice choice = plans ? plans->choices[r] : HeavyChoice{0, 0};
      const bool by_list = list && !list->items.empty();
      if (by_list || choice.tiles > 0) {
        // Short and medium lengths: the heaviest query tiles as one item per piece of the keys that they see (pieces of the
        // one block, or the ring blocks), with partial results; every other tile a whole item of the same launch that writes
        // its finished rows itself.  Then the merge of the cut rows, straight to the sequence-layout shards.
        const HeavyPieces hp = by_list ? list->hp : heavy_pieces(*p, choice.pieces);
        const void* kp[kMaxHeavyPieces];
        const void* vp[kMaxHeavyPieces];
        usp_posdesc pd[kMaxHeavyPieces];
        int lk[kMaxHeavyPieces];
        float* o_ptrs[kMaxHeavyPieces];
        float* l_ptrs[kMaxHeavyPieces];
        size_t held = 0;   // rows of partial results before this one
        for (int n = 0; n < hp.n; ++n) {
          const size_t row_off = (size_t)hp.first[n] * kv_pitch * p->hs * es;
          kp[n] = (const char*)kb[hp.block[n]] + row_off;
          // (transposed tiles: a piece begins hp.first / 64 tiles into every head's run of tiles)
          vp[n] = (const char*)vb[hp.block[n]] + (f.v_transposed ? (size_t)(hp.first[n] / 64) * p->hs * 64 * es : row_off);
          pd[n] = piece_of(kds[hp.block[n]], hp.first[n], hp.last[n]);
          lk[n] = (int)(hp.last[n] - hp.first[n]);
          if (by_list) {   // one behind the other
            o_ptrs[n] = (float*)(ws + f.o_parts) + held * hq * p->hs;
            l_ptrs[n] = (float*)(ws + f.lse_parts) + held * hq;
            held += (size_t)p->bs * (Lq - list->row0[n]);
          } else {
            o_ptrs[n] = (float*)(ws + f.o_parts + (size_t)n * f.part_o_bytes);
            l_ptrs[n] = (float*)(ws + f.lse_parts + (size_t)n * f.part_lse_bytes);
          }
        }
        MixedLaunch mixed = {(char*)o + group_off, lse_rank, by_list ? 0 : choice.tiles, f.v_transposed};
        if (by_list) {
          mixed.listed = list->items.data();
          mixed.n_listed = (int)list->items.size();
          mixed.part_row0 = list->row0;
        }
        st = launch_attn_fwd_partials((const char*)q + group_off, kp, vp, pd, lk, hp.n, o_ptrs, l_ptrs, p->bs, Lq, Lq, hq,
                                      hkv, p->hs, scale, p->causal ? 1 : 0, qd, stream, &seq, &mixed);
        if (st != USP_OK) return st;
        const RowTiles rows(qd, Lq, p->causal);
        const int64_t row0 = by_list ? list->merge_row0 : rows.begin(rows.n - choice.tiles);
        st = launch_lse_merge((const void* const*)o_ptrs, (const float* const*)l_ptrs, hp.n, (char*)o + group_off, lse_rank,
                              p->bs, Lq, hq, p->hs, USP_FP32, p->dtype, stream, &seq, row0, mixed.part_row0);
        if (st != USP_OK) return st;
        continue;
      }
      const int splits = key_splits(*p);
      if (splits > 0) {
        // Short sequence: every block in `splits` pieces, each (query tile, head, piece) its own work item of one
        // launch; the pieces' partial results are merged, and O takes the separate pass back to the sequence layout.
        const int64_t piece = ((Lq + splits - 1) / splits + 63) / 64 * 64;
        const void* kp[USP_MAX_RING_BLOCKS];
        const void* vp[USP_MAX_RING_BLOCKS];
        usp_posdesc pd[USP_MAX_RING_BLOCKS];
        int lk[USP_MAX_RING_BLOCKS];
        float* o_ptrs[USP_MAX_RING_BLOCKS];
        float* l_ptrs[USP_MAX_RING_BLOCKS];
        int n = 0;
        for (int i = 0; i < R; ++i)
          for (int64_t a0 = 0; a0 < Lq; a0 += piece, ++n) {
            const int64_t a1 = std::min(Lq, a0 + piece);
            const size_t row_off = (size_t)a0 * kv_pitch * p->hs * es;
            kp[n] = (const char*)kb[i] + row_off;
            vp[n] = (const char*)vb[i] + row_off;
            pd[n] = piece_of(kds[i], a0, a1);
            lk[n] = (int)(a1 - a0);
            o_ptrs[n] = (float*)(ws + f.o_parts + (size_t)n * f.part_o_bytes);
            l_ptrs[n] = (float*)(ws + f.lse_parts + (size_t)n * f.part_lse_bytes);
          }
        st = launch_attn_fwd_partials((const char*)q + group_off, kp, vp, pd, lk, n, o_ptrs, l_ptrs, p->bs, Lq, Lq, hq,
                                      hkv, p->hs, scale, p->causal ? 1 : 0, qd, stream, &seq);
        if (st != USP_OK) return st;
        // the merge writes O straight to the sequence-layout shards (step 6 rides on its stores)
        st = launch_lse_merge((const void* const*)o_ptrs, (const float* const*)l_ptrs, n, (char*)o + group_off, lse_rank,
                              p->bs, Lq, hq, p->hs, USP_FP32, p->dtype, stream, &seq);
        if (st != USP_OK) return st;
        continue;
      }
      st = launch_ring_attn_fwd((const char*)q + group_off, kb, vb, kds, R, (char*)o + group_off, lse_rank, p->bs, Lq,
                                Lq, hq, hkv, p->hs, scale, p->causal ? 1 : 0, qd, p->dtype, p->dtype, stream, &seq,
                                nullptr, f.v_transposed);
      if (st != USP_OK) return st;
      continue;
    }
    const void* o_ptrs[USP_MAX_MERGE_PARTS];
    const float* l_ptrs[USP_MAX_MERGE_PARTS];
    if (R > USP_MAX_MERGE_PARTS) return USP_ERR_UNSUPPORTED;
    for (int i = 0; i < R; ++i) {
      const int s = ((r - i) % R + R) % R;
      usp_posdesc kd;
      usp_local_positions(p, s, u, nullptr, &kd);
      void* o_dst = R > 1 ? (void*)(ws + f.o_parts + (size_t)i * f.part_o_bytes) : (void*)(ws + f.o_head);
      float* l_dst = R > 1 ? (float*)(ws + f.lse_parts + (size_t)i * f.part_lse_bytes) : lse_rank;
      st = launch_block_attn_fwd(ws + f.q_head, k_block(s, u), v_block(s, u), o_dst, l_dst, p->bs, Lq,
                                 Lq, hq, hkv, p->hs, scale, p->causal ? 1 : 0, qd, kd, p->dtype,
                                 R > 1 ? USP_FP32 : p->dtype, stream);
      if (st != USP_OK) return st;
      o_ptrs[i] = o_dst;
      l_ptrs[i] = l_dst;
    }
    if (R > 1) {
      // Step 6 rides on the merge's stores: O goes straight to the sequence-layout shards of the Ulysses group
      const SeqLayoutIO seq = {(int)(p->L / N), p->hc, u * hq};
      const size_t group_off = (size_t)r * U * p->bs * (p->L / N) * p->hc * p->hs * es;
      st = launch_lse_merge(o_ptrs, l_ptrs, R, (char*)o + group_off, lse_rank, p->bs, Lq, hq, p->hs, USP_FP32, p->dtype,
                            stream, &seq);
      if (st != USP_OK) return st;
      continue;
    }
    // Step 6: O back to the sequence layout.
    st = launch_layout_a2a(*p, p->hc, USP_HEAD_TO_SEQ, ws + f.o_head, o, rank, rank + 1, rank, stream);
    if (st != USP_OK) return st;
  }
  return USP_OK;
}
}  // namespace

extern "C" int usp_attn_fwd(const usp_problem* p, const void* q, const void* k, const void* v, void* o, float* lse,
                            int rank_begin, int rank_end, void* workspace, size_t workspace_bytes, void* stream) try {
  return attn_fwd_impl(p, q, k, v, o, lse, rank_begin, rank_end, workspace, workspace_bytes, stream);
} catch (...) {
  return USP_ERR_LAUNCH;
}

// ---------------------------------------------------------------------------------------------
// usp_attn_fwd for callers that cannot allocate: the workspace is a static device array.  Each GPU the library
// runs on holds its own copy of the array (at its own address) until the process ends; host code never uses the
// array's name as an address, only what hipGetSymbolAddress returned for the current device.
// ---------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[USP_NOALLOC_SCRATCH_BYTES];

namespace {
// Device address of `scratch` on the current device (asked once per device), or null.
void* scratch_on_current_device() {
  static std::atomic<void*> known[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  void* ptr = known[dev].load(std::memory_order_acquire);
  if (!ptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    known[dev].store(ptr, std::memory_order_release);   // two threads that meet here store the same address
  }
  return ptr;
}
}  // namespace

extern "C" int usp_attn_fwd_noalloc(const usp_problem* p, const void* q, const void* k, const void* v, void* o,
                                    float* lse, int rank_begin, int rank_end, void* stream) try {
  int st = usp_validate(p);
  if (st != USP_OK) return st;
  const int N = p->ulysses * p->ring;
  if (rank_begin < 0 || rank_end > N || rank_begin >= rank_end) return USP_ERR_UNSUPPORTED;
  int c0, c1;
  column_range(*p, rank_begin, rank_end, &c0, &c1);
  // the partial results of a cut of the heaviest tiles are optional: without room for them the launch stays whole
  const bool heavy_fits = plan_fwd(*p, c1 - c0, true).total <= USP_NOALLOC_SCRATCH_BYTES;
  if (!heavy_fits && plan_fwd(*p, c1 - c0, false).total > USP_NOALLOC_SCRATCH_BYTES) return USP_ERR_WORKSPACE;   // beyond the static array
  void* ptr = scratch_on_current_device();
  if (!ptr) return USP_ERR_LAUNCH;
  // every region of the workspace is written by a kernel of the call before a kernel reads it: nothing to clear
  return attn_fwd_impl(p, q, k, v, o, lse, rank_begin, rank_end, ptr, USP_NOALLOC_SCRATCH_BYTES, stream, heavy_fits);
} catch (...) {
  return USP_ERR_LAUNCH;
}

extern "C" int usp_attn_delta(const void* o, const void* d_o, float* delta, int bs, int64_t L, int h, int hs,
                              void* stream) {
  if (!o || !d_o || !delta) return USP_ERR_NULL;
  if (bs < 1 || L < 1 || h < 1) return USP_ERR_SHAPE;
  if (hs != 64 && hs != 128) return USP_ERR_UNSUPPORTED;
  if (L >= (int64_t)1 << 31) return USP_ERR_UNSUPPORTED;
  const PrepareTensor t = {d_o, o, nullptr, delta, 1, 0, 1, 0, 1, h, h};
  return launch_bwd_prepare(&t, 1, bs, L, hs, (hipStream_t)stream);
}

extern "C" int usp_block_attn_bwd(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                                  const float* delta, float* dq, float* dk, float* dv, int bs, int64_t Lq, int64_t Lk,
                                  int hq, int hkv, int hs, float scale, int causal, const usp_posdesc* qpos,
                                  const usp_posdesc* kpos, int accumulate, void* stream) try {
  if (!q || !k || !v || !d_o || !lse || !delta || !dq || !dk || !dv) return USP_ERR_NULL;
  if (bs < 1 || Lq < 1 || Lk < 1 || hq < 1 || hkv < 1) return USP_ERR_SHAPE;
  if (hq % hkv) return USP_ERR_DEGREE;
  if (hs != 64 && hs != 128) return USP_ERR_UNSUPPORTED;
  if (!(scale >= 0.0f) || isinf(scale)) return USP_ERR_UNSUPPORTED;
  if (Lq >= (int64_t)1 << 31 || Lk >= (int64_t)1 << 31) return USP_ERR_UNSUPPORTED;
  usp_posdesc qd = {0, Lq, 0, 0}, kd = {0, Lk, 0, 0};
  if (causal) {
    if (!qpos || !kpos) return USP_ERR_NULL;
    if (!desc_ok(qpos, Lq) || !desc_ok(kpos, Lk)) return USP_ERR_SHAPE;
    qd = *qpos;
    kd = *kpos;
  }
  if (scale == 0.0f) scale = 1.0f / sqrtf((float)hs);
  return launch_block_attn_bwd(q, k, v, d_o, lse, delta, dq, dk, dv, bs, Lq, Lk, hq, hkv, hs, scale, causal ? 1 : 0,
                               qd, kd, accumulate ? 1 : 0, accumulate ? 1 : 0, (hipStream_t)stream);
} catch (...) {
  return USP_ERR_LAUNCH;
}

// ---------------------------------------------------------------------------------------------
// Algorithm 1 backward.  Workspace plan:
//   q_head, do_head         : one rank's Q and dO, [bs][head][row][hs] (reused rank after rank); O is read once, for D_i,
//                             straight from the sequence-layout shards;
//   (with Ulysses degree 1 a rank's Q, dO and every K/V block lie in the sequence-layout shards as they are wanted: these
//   four regions are empty and the kernels read the caller's tensors where they are)
//   delta                   : one rank's D_i;
//   k_head, v_head          : every K/V block of the columns in range, [bs][head][row][hs];
//   dq_acc                  : one rank's fp32 dQ;  dk_acc, dv_acc : fp32, one per K/V block; each in as many copies as the
//                             cut has slices.  Unused where results leave the kernels as bf16.
// All ranks at once (see there): D_i of all of them from q_head on, in the room up to the accumulators.
// ---------------------------------------------------------------------------------------------
namespace {

struct BwdPlan {
  size_t q_head, do_head, delta, k_head, v_head, dq_acc, dk_acc, dv_acc, total;
  size_t kv_block_bytes, kv_acc_bytes;   // kv_acc_bytes: ALL copies of one block's dk (or dv) accumulator
  BwdCopies copies;                      // how the launch pairs are cut, and the copies of dq / dk / dv they fill
  int dkdv_copies;
  size_t ds, ds_bytes;                   // room for the dS of one launch pair (used when the workspace reaches that far)
  size_t total_with_ds;
};

BwdPlan plan_bwd(const usp_problem& p, int n_cols) {
  BwdPlan f;
  const size_t es = dtype_size(p.dtype);
  const size_t Lq = p.L / p.ring, hq = p.hc / p.ulysses, hkv = p.hk / p.ulysses;
  const size_t q_elems = (size_t)p.bs * Lq * hq * p.hs, kv_elems = (size_t)p.bs * Lq * hkv * p.hs;
  const size_t qb = up256(q_elems * es);
  f.kv_block_bytes = kv_elems * es;   // exact: blocks are packed back to back
  // every launch pair of this problem is cut the same way (that of its largest launch: up to 16 blocks)
  f.copies.cut = plan_bwd_cut(p.bs, (int64_t)Lq, (int64_t)Lq, (int)hq, (int)hkv, std::min(p.ring, USP_MAX_RING_BLOCKS), true, !p.causal);
  f.copies.dq_stride = q_elems;
  f.copies.dkdv_stride = kv_elems;
  f.dkdv_copies = (int)(hq / hkv) / f.copies.cut.heads_per_wg * f.copies.cut.q_splits;
  f.kv_acc_bytes = up256(kv_elems * sizeof(float) * f.dkdv_copies);
  const size_t blocks = (size_t)p.ring * n_cols;
  size_t off = 0;
  const bool in_place = p.ulysses == 1;
  f.q_head = off; off += in_place ? 0 : qb;
  f.do_head = off; off += in_place ? 0 : qb;
  f.delta = off; off += up256((size_t)p.bs * hq * Lq * sizeof(float));
  f.k_head = off; off += in_place ? 0 : up256(f.kv_block_bytes * blocks);
  f.v_head = off; off += in_place ? 0 : up256(f.kv_block_bytes * blocks);
  f.dq_acc = off; off += up256(q_elems * sizeof(float) * f.copies.cut.k_splits);
  f.dk_acc = off; off += f.kv_acc_bytes * blocks;
  f.dv_acc = off; off += f.kv_acc_bytes * blocks;
  f.total = off;
  f.ds = off;
  // dS is kept only at head size 128: at 64 forming S and dP a second time costs less than moving 4 bytes per pair
  // (measured: 2.32 ms recomputed against 2.46 ms with dS kept on the Ulysses-8 rank of L = 32768)
  f.ds_bytes = bwd_keeps_ds(p.hs) ? up256(bwd_ds_bytes(p.bs, (int64_t)Lq, (int64_t)Lq, (int)hq, std::min(p.ring, USP_MAX_RING_BLOCKS))) : 0;
  f.total_with_ds = off + f.ds_bytes;
  return f;
}

// How the launch pair of ring rank r (r < 0: of all ranks at once) is cut: within what the workspace was sized for (`most`),
// the number of slices and of heads per item under which the pair ends first.  dQ items fill the gaps behind the dK/dV items,
// so that long sequences need no slices where the two kernels on their own took two to four of each, and every slice
// saved is a copy of the outputs less.  Worked out by playing the launch through, as work_out_heavy_choice() does for the
// forward: 10 us per dQ item and 1.2 per 32 of its keys, 6 and 1.68 per 32 queries of a dK/dV item (0.62 of these at head
// size 64), the copies at 4.5 TB/s and 6 us for their launch.  Against 130 measured cuts of eleven problems, L = 2048 to
// 16384, this is off by 6 % on average and picks a cut within 0.3 % of the best one (one of eight Ulysses ranks of L = 8192:
// 4 + 4 slices 298 us, 2 + 2 279; 32 heads of L = 2048: 2 + 2 slices 217 us, none 168).  What is played is not in every
// zigzag ring what is launched: every block's tiles are taken as RowTiles has them and as many as the first ring row's,
// where the launch cuts all blocks alike (common_row_tiles: a whole ring in a row) and takes the blocks in ring order.  One
// zigzag problem in ten is then cut otherwise; playing the very launch was no better on these (35 measured: 2.3 % slower on
// average, 0.76 to 1.07 x), the model is not that fine.
BwdCut work_out_bwd_cut(const usp_problem& p, int r, const BwdCut& most) {
  const int64_t Lq = p.L / p.ring;
  const int hq = r < 0 ? p.hc : p.hc / p.ulysses, hkv = r < 0 ? p.hk : p.hk / p.ulysses, g = hq / hkv;
  const int q_first = r < 0 ? 0 : r, q_last = r < 0 ? p.ring - 1 : r;
  BwdCut best = most;
  if (r < 0) best.k_splits = 1;   // dQ leaves as bf16
  const int m = p.bs * hkv;       // KV groups: alike, so one of them is played, on its share of the CUs
  if ((Lq + 255) / 256 * (q_last - q_first + 1) * m * g > 8 * kPlanCUs) return best;   // items to spare
  const int cus = std::max(1, (kPlanCUs + m / 2) / m);
  // 32-key steps of every (ring row, query tile), 32-query steps of every (K/V block, key tile): under kpos <= qpos the
  // keys that a run of queries sees are a prefix of each run of keys, the queries that see a key a suffix of theirs
  std::vector<usp_posdesc> pos(p.ring);
  std::vector<RowTiles> tiles;
  for (int s = 0; s < p.ring; ++s) {
    ring_block_desc(p, s, &pos[s]);
    tiles.emplace_back(pos[s], Lq, p.causal);
  }
  const int T = tiles[0].n;   // (the ring row whose runs adjoin may have one less: it is charged the one more)
  std::vector<double> dq, dkdv;
  auto steps = [](int64_t n) { return (double)((n + 31) / 32); };
  for (int t = T - 1; t >= 0; --t)
    for (int i = q_first; i <= q_last; ++i) {
      const int64_t last = pos_max(pos[i], tiles[i].begin(t), tiles[i].end(t));
      double w = 0.0;
      for (const usp_posdesc& k : pos)
        w += p.causal ? steps(std::clamp<int64_t>(last - k.start0 + 1, 0, k.len0)) + steps(std::clamp<int64_t>(last - k.start1 + 1, 0, k.len1)) : steps(Lq);
      dq.push_back(w);
    }
  for (int s = 0; s < p.ring; ++s)
    for (int t = 0; t < T; ++t) {
      const int64_t first = pos_min(pos[s], tiles[s].begin(t), tiles[s].end(t));
      double w = 0.0;
      for (int i = q_first; i <= q_last; ++i)
        w += p.causal ? steps(pos[i].len0 - std::clamp<int64_t>(first - pos[i].start0, 0, pos[i].len0)) +
                            steps(pos[i].len1 - std::clamp<int64_t>(first - pos[i].start1, 0, pos[i].len1))
                      : steps(Lq);
      dkdv.push_back(w);
    }
  const double f = p.hs == 128 ? 1.0 : 0.62, tq = 1.2 * f, tk = 1.68 * f;
  double sum_q = 0.0, sum_k = 0.0, max_q = 0.0, max_k = 0.0;
  for (double w : dq) { sum_q += w; max_q = std::max(max_q, w); }
  for (double w : dkdv) { sum_k += w; max_k = std::max(max_k, w); }
  std::vector<double> free_at;   // the workgroups' finish times, a min-heap
  double best_us = 1e30;
  auto consider = [&](const BwdCut& c, double factor) {
    const int parts = g / c.heads_per_wg * c.q_splits;   // dK/dV items per key tile, copies of dK and dV
    const double copied = (c.k_splits > 1 ? (double)c.k_splits * hq * (q_last - q_first + 1) : 0.0) + (parts > 1 ? 2.0 * parts * hkv * p.ring : 0.0);
    const double copies_us = copied > 0.0 ? 6.0 + copied * p.bs * Lq * p.hs * 4.0 / 4.5e6 : 0.0;
    const double limit = best_us / factor - copies_us;   // it has to end before this
    const double item_k = tk * c.heads_per_wg / c.q_splits, item_q = tq / c.k_splits;
    const double share = (parts * (6.0 * dkdv.size() + item_k * sum_k) + g * c.k_splits * (10.0 * dq.size() + item_q * sum_q)) / cus;
    if (std::max({share, 6.0 + item_k * max_k, 10.0 + item_q * max_q}) >= limit) return;   // most cuts end here, unplayed
    free_at.assign(cus, 0.0);
    double end = 0.0;
    auto play = [&](double us, int times) {
      for (int i = 0; i < times; ++i) {
        const double t = free_at[0] + us;
        end = std::max(end, t);
        int at = 0;   // the first to be free takes the item; its new time sinks to its place
        for (int kid; (kid = 2 * at + 1) < cus; at = kid) {
          if (kid + 1 < cus && free_at[kid + 1] < free_at[kid]) ++kid;
          if (free_at[kid] >= t) break;
          free_at[at] = free_at[kid];
        }
        free_at[at] = t;
      }
      return end < limit;
    };
    for (double w : dkdv)
      if (!play(6.0 + item_k * w, parts)) return;
    for (double w : dq)
      if (!play(10.0 + item_q * w, g * c.k_splits)) return;
    best_us = factor * (end + copies_us);
    best = c;
  };
  // (what the workspace was sized for is left for a gain of 3 % or more: at L = 32768 cuts that look alike here differ by 1 %)
  consider(best, 0.97);
  const int max_copies = g / most.heads_per_wg * most.q_splits;
  const int max_slices = (int)std::clamp<int64_t>(Lq / 512, 1, 4), max_k_splits = best.k_splits;
  for (int h = g; h >= 1; --h)
    for (int q = 1; g % h == 0 && q <= max_slices && g / h * q <= max_copies; q *= 2)
      for (int k = 1; k <= max_k_splits; k = k < 2 ? 2 : k + 2) consider(BwdCut{h, k, q}, 1.0);
  return best;
}

// Playing the cuts of a problem through takes the host 0.1 ms, 0.7 at most: the last answers are kept, as plans_of() keeps its.
BwdCut bwd_cut(const usp_problem& p, int r, const BwdCut& most) {
  struct Entry { usp_problem p; int r; BwdCut cut; };   // (`most` follows from the problem)
  static std::mutex mu;
  static std::vector<Entry> seen;
  std::lock_guard<std::mutex> lock(mu);
  for (const Entry& e : seen)
    if (e.r == r && same_problem(e.p, p)) return e.cut;
  if (seen.size() >= 256) seen.erase(seen.begin());
  seen.push_back(Entry{p, r, work_out_bwd_cut(p, r, most)});
  return seen.back().cut;
}

}  // namespace

extern "C" size_t usp_attn_bwd_workspace_bytes(const usp_problem* p, int n_ranks) {
  if (usp_validate(p) != USP_OK || n_ranks < 1 || p->dtype != USP_BF16) return 0;
  const int cols = n_ranks == 1 ? 1 : p->ulysses;
  return plan_bwd(*p, cols).total;
}

extern "C" size_t usp_attn_bwd_workspace_bytes_with_ds(const usp_problem* p, int n_ranks) {
  if (usp_validate(p) != USP_OK || n_ranks < 1 || p->dtype != USP_BF16) return 0;
  const int cols = n_ranks == 1 ? 1 : p->ulysses;
  return plan_bwd(*p, cols).total_with_ds;
}

extern "C" int usp_attn_bwd(const usp_problem* p, const void* q, const void* k, const void* v, const void* o,
                            const float* lse, const void* d_o, void* dq, void* dk, void* dv, int rank_begin,
                            int rank_end, void* workspace, size_t workspace_bytes, void* stream_) try {
  int st = usp_validate(p);
  if (st != USP_OK) return st;
  if (p->dtype != USP_BF16) return USP_ERR_DTYPE;
  if (!q || !k || !v || !o || !lse || !d_o || !dq || !dk || !dv) return USP_ERR_NULL;
  const int U = p->ulysses, R = p->ring, N = U * R;
  if (rank_begin < 0 || rank_end > N || rank_begin >= rank_end) return USP_ERR_UNSUPPORTED;
  int c0, c1;
  column_range(*p, rank_begin, rank_end, &c0, &c1);
  const int n_cols = c1 - c0;
  BwdPlan f = plan_bwd(*p, n_cols);
  if (!workspace || workspace_bytes < f.total) return USP_ERR_WORKSPACE;
  if ((uintptr_t)workspace & 255) return USP_ERR_WORKSPACE;
  hipStream_t stream = (hipStream_t)stream_;
  char* ws = (char*)workspace;
  if (f.ds_bytes && workspace_bytes >= f.total_with_ds) f.copies.ds = ws + f.ds;   // room to keep dS between the two kernels
  const int64_t Lq = p->L / R;
  const int hq = p->hc / U, hkv = p->hk / U;
  const float scale = p->scale == 0.0f ? 1.0f / sqrtf((float)p->hs) : p->scale;
  const size_t q_elems = (size_t)p->bs * Lq * hq * p->hs, kv_elems = (size_t)p->bs * Lq * hkv * p->hs;
  const size_t es = dtype_size(p->dtype);
  auto slot = [&](int r, int u) { return (size_t)r * n_cols + (u - c0); };
  if ((size_t)R * n_cols > USP_MAX_MERGE_PARTS) return USP_ERR_UNSUPPORTED;

  // Results may only be written while inputs are still read if they share no memory.
  const size_t q_all = q_elems * N * es, kv_all = kv_elems * N * es;
  bool apart = true;
  {
    const void* const in[] = {q, k, v, o, d_o, lse};
    const size_t in_bytes[] = {q_all, kv_all, kv_all, q_all, q_all, (size_t)p->bs * Lq * hq * N * sizeof(float)};
    const void* const out[] = {dq, dk, dv};
    const size_t out_bytes[] = {q_all, kv_all, kv_all};
    for (int i = 0; i < 6; ++i)
      for (int j = 0; j < 3; ++j)
        if (overlap(in[i], in_bytes[i], out[j], out_bytes[j])) apart = false;
  }
  // With Ulysses degree 1 the all-to-alls are the identity; with a batch of one the shards of a ring row are contiguous,
  // [Lq][heads][hs].  Either way a rank's tensors are its heads of the ring row's rows.
  const bool seq_rows = U == 1 || p->bs == 1;
  const bool direct = seq_rows && apart && R <= USP_MAX_RING_BLOCKS;   // results may leave the kernels as bf16, to their place
  const double rank_us = 10.0 * p->hs * p->bs * hq * (double)Lq * (double)p->L * (p->causal ? 0.5 : 1.0) / 0.8e9;
  auto q_at = [&](const void* t, int r, int u) { return (char*)t + ((size_t)r * p->bs * Lq * p->hc + (size_t)u * hq) * p->hs * es; };
  auto kv_at = [&](const void* t, int r, int u) { return (char*)t + ((size_t)r * p->bs * Lq * p->hk + (size_t)u * hkv) * p->hs * es; };
  usp_posdesc ring_pos[USP_MAX_MERGE_PARTS];   // positions of every ring row
  for (int r = 0; r < R; ++r) usp_local_positions(p, r, 0, nullptr, &ring_pos[r]);

  // Every rank at once: in place, the tensors of all ranks are one dense problem of R query blocks, R key blocks and all
  // heads, which go through ONE launch instead of one (and conversions) per rank.  Not where dS is kept and a rank is long
  // enough to gain by that.  Measured, with dS kept rank by rank / all at once, 32/8 heads, U 2 x R 2: 107 us per rank (by
  // the estimate above) 876 / 505 us, 328 1813 / 1402, 429 2070 / 1834, 966 4042 / 3889, 1717 6484 / 6887; MHA, U 2 x R 4:
  // 483 4937 / 3998, 858 7674 / 6906.  (The two meet near 1 ms; the line lies lower.)
  const bool aligned = (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o | (uintptr_t)d_o) & 15) == 0;
  if (direct && aligned && N > 1 && rank_begin == 0 && rank_end == N) {
    BwdCopies c;
    c.cut = bwd_cut(*p, -1, f.copies.cut);
    const int copies = p->hc / p->hk / c.cut.heads_per_wg * c.cut.q_splits;
    const size_t delta_bytes = up256(q_elems / p->hs * N * sizeof(float));   // in the room from q_head up to the accumulators
    if ((!f.copies.ds || rank_us < 400.0) && delta_bytes <= f.dk_acc - f.q_head) {
      const size_t kv_block = kv_elems * U;   // elements of a ring row, all heads
      c.dq_stride = 0;
      c.dkdv_stride = kv_block;
      const bool dkdv_bf16 = copies == 1;
      float* delta = (float*)(ws + f.q_head);
      const PrepareTensor d = {d_o, o, nullptr, delta, 1, 0, R, 0, 1, p->hc, p->hc};
      st = launch_bwd_prepare(&d, 1, p->bs, Lq, p->hs, stream);
      if (st != USP_OK) return st;
      const void *kb[USP_MAX_RING_BLOCKS], *vb[USP_MAX_RING_BLOCKS];
      float *dkb[USP_MAX_RING_BLOCKS], *dvb[USP_MAX_RING_BLOCKS];
      const int acc[USP_MAX_RING_BLOCKS] = {0};
      for (int s = 0; s < R; ++s) {
        kb[s] = kv_at(k, s, 0);
        vb[s] = kv_at(v, s, 0);
        dkb[s] = dkdv_bf16 ? (float*)kv_at(dk, s, 0) : (float*)(ws + f.dk_acc) + (size_t)s * copies * kv_block;
        dvb[s] = dkdv_bf16 ? (float*)kv_at(dv, s, 0) : (float*)(ws + f.dv_acc) + (size_t)s * copies * kv_block;
      }
      const BwdPlace io = {{Lq * p->hc, p->hc, 1}, {Lq * p->hk, p->hk, 1}, p->hc, dkdv_bf16 ? p->hk : 0, R, ring_pos};
      st = launch_ring_attn_bwd(q, kb, vb, ring_pos, R, d_o, lse, delta, (float*)dq, dkb, dvb, p->bs, Lq, Lq,
                                p->hc, p->hk, p->hs, scale, p->causal ? 1 : 0, ring_pos[0], 0, acc, stream, &c, &io);
      if (st != USP_OK || dkdv_bf16) return st;
      ConvertTensor t[2];
      for (int i = 0; i < 2; ++i) {
        t[i].src = i ? dvb[0] : dkb[0];
        t[i].dst = i ? dv : dk;
        t[i].n = t[i].copy_stride = t[i].dst_blk = kv_block;
        t[i].n_copies = copies;
        t[i].n_blocks = R;
        t[i].src_blk = kv_block * copies;
      }
      return launch_bwd_convert(t, 2, p->dtype, stream);
    }
  }

  // Otherwise rank after rank.  Ulysses degree 1: everything is read in place.  Else Q, dO, K and V are staged in head
  // layout, in the launch that forms D_i, also where a batch of one could be read in place: rows as far apart as the whole
  // model's heads are long (8 KiB) cost the dK/dV kernel 2.4 %, more than the copies (L = 32768: 1837 -> 1882 us).
  const bool in_place = U == 1;
  const RowPlace place_q = in_place ? RowPlace{Lq * hq, hq, 1} : RowPlace{Lq * hq, 1, (int)Lq};
  const RowPlace place_kv = in_place ? RowPlace{Lq * hkv, hkv, 1} : RowPlace{Lq * hkv, 1, (int)Lq};

  // first contribution to a K/V block overwrites its accumulator, later ones add
  bool touched[USP_MAX_MERGE_PARTS] = {false};

  const bool one_rank = rank_end - rank_begin == 1;
  BwdCopies run = f.copies;
  // one cut for all ranks of the call, which add to the same copies: that of the first one's ring row (with dS kept the two
  // kernels run one after the other)
  if (!run.ds) run.cut = bwd_cut(*p, rank_begin / U, run.cut);
  const int dkdv_copies = hq / hkv / run.cut.heads_per_wg * run.cut.q_splits;
  const bool dq_bf16 = direct && run.cut.k_splits == 1;
  const bool dkdv_bf16 = direct && one_rank && dkdv_copies == 1;
  const BwdPlace place = {place_q, place_kv, dq_bf16 ? p->hc : 0, dkdv_bf16 ? p->hk : 0, 1, nullptr};
  SeqLayoutIO seq_q = {(int)(p->L / N), p->hc, 0};
  ConvertTensor convert[3];
  int n_convert = 0;
  for (int rank = rank_begin; rank < rank_end; ++rank) {
    const int r = rank / U, u = rank % U;
    const char* q_rank = in_place ? q_at(q, r, u) : ws + f.q_head;
    const char* do_rank = in_place ? q_at(d_o, r, u) : ws + f.do_head;
    seq_q.head0 = u * hq;
    const size_t group_off = (size_t)r * U * p->bs * (p->L / N) * p->hc * p->hs * es;   // the Ulysses group's first shard
    float* delta = (float*)(ws + f.delta);
    {
      // D_i of this rank's rows, and what has to be staged: its Q and dO, and once, the K/V blocks of every ring row
      PrepareTensor t[4] = {{d_o, o, in_place ? nullptr : ws + f.do_head, delta, U, r, 1, u, 1, p->hc, hq},
                            {q, nullptr, ws + f.q_head, nullptr, U, r, 1, u, 1, p->hc, hq},
                            {k, nullptr, ws + f.k_head, nullptr, U, 0, R, c0, n_cols, p->hk, hkv},
                            {v, nullptr, ws + f.v_head, nullptr, U, 0, R, c0, n_cols, p->hk, hkv}};
      st = launch_bwd_prepare(t, in_place ? 1 : rank == rank_begin ? 4 : 2, p->bs, Lq, p->hs, stream);
      if (st != USP_OK) return st;
    }
    const float* lse_rank = lse + (size_t)rank * p->bs * hq * Lq;
    // The ring loop of this rank, step i on block s = (r - i) mod R: up to USP_MAX_RING_BLOCKS steps per launch
    // pair (a dQ item keeps its accumulator in registers across them, the dK/dV items are spread over them).  dQ adds
    // after the first launch of this rank; a block's dK/dV add after the first rank that touched it.  Blocks that lie
    // wholly behind the rank's rows (contiguous split, causal) are left out where an absent block costs nothing: not where
    // the kernels write dK/dV themselves, zeros then included.
    int steps[USP_MAX_MERGE_PARTS], n_steps = 0;
    for (int i = 0; i < R; ++i) {
      const int s = ((r - i) % R + R) % R;
      if (dkdv_bf16 || !p->causal || pos_min(ring_pos[s], 0, Lq) <= pos_max(ring_pos[r], 0, Lq)) steps[n_steps++] = s;
    }
    for (int i0 = 0; i0 < n_steps; i0 += USP_MAX_RING_BLOCKS) {
      const int nb = n_steps - i0 < USP_MAX_RING_BLOCKS ? n_steps - i0 : USP_MAX_RING_BLOCKS;
      const void* kb[USP_MAX_RING_BLOCKS];
      const void* vb[USP_MAX_RING_BLOCKS];
      float* dkb[USP_MAX_RING_BLOCKS];
      float* dvb[USP_MAX_RING_BLOCKS];
      usp_posdesc kds[USP_MAX_RING_BLOCKS];
      int acc[USP_MAX_RING_BLOCKS];
      for (int j = 0; j < nb; ++j) {
        const int s = steps[i0 + j];
        kds[j] = ring_pos[s];
        const size_t sl = slot(s, u);
        kb[j] = in_place ? kv_at(k, s, u) : ws + f.k_head + sl * f.kv_block_bytes;
        vb[j] = in_place ? kv_at(v, s, u) : ws + f.v_head + sl * f.kv_block_bytes;
        dkb[j] = (float*)(dkdv_bf16 ? kv_at(dk, s, u) : ws + f.dk_acc + sl * f.kv_acc_bytes);
        dvb[j] = (float*)(dkdv_bf16 ? kv_at(dv, s, u) : ws + f.dv_acc + sl * f.kv_acc_bytes);
        acc[j] = touched[sl] ? 1 : 0;
        touched[sl] = true;
      }
      st = launch_ring_attn_bwd(q_rank, kb, vb, kds, nb, do_rank, lse_rank, delta,
                                (float*)(dq_bf16 ? q_at(dq, r, u) : ws + f.dq_acc), dkb, dvb, p->bs, Lq, Lq, hq, hkv, p->hs,
                                scale, p->causal ? 1 : 0, ring_pos[r], i0 > 0 ? 1 : 0, acc, stream, &run, &place);
      if (st != USP_OK) return st;
    }
    // dQ of this rank: the copies summed, converted and written straight to the sequence-layout shards of its Ulysses
    // group (the reverse all-to-all rides on the conversion's stores)
    if (!dq_bf16) {
      ConvertTensor& t = convert[n_convert++];
      t.src = (const float*)(ws + f.dq_acc);
      t.dst = (char*)dq + group_off;
      t.n = t.copy_stride = q_elems;
      t.n_copies = run.cut.k_splits;
      t.seq = &seq_q;
      t.bs = p->bs; t.rows = Lq; t.heads = hq; t.hs = p->hs;
      if (!one_rank) {   // the next rank uses the accumulator
        st = launch_bwd_convert(convert, n_convert, p->dtype, stream);
        if (st != USP_OK) return st;
        n_convert = 0;
      }
    }
  }

  // dK, dV of every block the range touched: all ring rows of the columns whose ranks were run.  A range that
  // straddles ring rows without covering every column (say [U-1, U+1)) leaves columns between c0 and c1 unvisited:
  // their accumulators were never written, and their head slices of dk / dv stay as the caller left them.
  // The copies are summed, converted and written straight to the blocks' sequence-layout shards; a single rank's in one
  // launch with its dQ.
  if (!dkdv_bf16)
    for (int u = c0; u < c1; ++u) {
      uint64_t absent = 0;   // ring rows that no rank of the range sees: zeros
      for (int s = 0; s < R; ++s)
        if (!touched[slot(s, u)]) absent |= 1ull << s;
      if (absent == ~0ull >> (64 - R)) continue;   // (every rank sees its own block)
      const SeqLayoutIO seq_u = {(int)(p->L / N), p->hk, u * hkv};
      for (int i = 0; i < 2; ++i) {
        ConvertTensor& t = convert[n_convert++];
        t.src = (const float*)(ws + (i ? f.dv_acc : f.dk_acc) + slot(0, u) * f.kv_acc_bytes);
        t.dst = i ? dv : dk;
        t.n = t.copy_stride = kv_elems;
        t.n_copies = dkdv_copies;
        t.n_blocks = R;
        t.absent = absent;
        t.src_blk = n_cols * f.kv_acc_bytes / sizeof(float);
        t.dst_blk = kv_elems * U;
        t.seq = &seq_u;
        t.bs = p->bs; t.rows = Lq; t.heads = hkv; t.hs = p->hs;
      }
      st = launch_bwd_convert(convert, n_convert, p->dtype, stream);
      if (st != USP_OK) return st;
      n_convert = 0;
    }
  return n_convert ? launch_bwd_convert(convert, n_convert, p->dtype, stream) : USP_OK;
} catch (...) {
  return USP_ERR_LAUNCH;
}

extern "C" int usp_ring_attn_bwd(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                                 const usp_posdesc* kpos_blocks, int n_blocks, const void* d_o, const float* lse,
                                 const float* delta, float* dq, float* const* dk_blocks, float* const* dv_blocks,
                                 int bs, int64_t Lq, int64_t Lk, int hq, int hkv, int hs, float scale, int causal,
                                 const usp_posdesc* qpos, int accumulate_dq, const int* accumulate_dkdv,
                                 void* stream) try {
  if (!q || !k_blocks || !v_blocks || !d_o || !lse || !delta || !dq || !dk_blocks || !dv_blocks || !accumulate_dkdv)
    return USP_ERR_NULL;
  if (n_blocks < 1 || n_blocks > USP_MAX_RING_BLOCKS) return USP_ERR_UNSUPPORTED;
  if (bs < 1 || Lq < 1 || Lk < 1 || hq < 1 || hkv < 1) return USP_ERR_SHAPE;
  if (hq % hkv) return USP_ERR_DEGREE;
  if (hs != 64 && hs != 128) return USP_ERR_UNSUPPORTED;
  if (!(scale >= 0.0f) || isinf(scale)) return USP_ERR_UNSUPPORTED;
  if (Lq >= (int64_t)1 << 31 || Lk >= (int64_t)1 << 31) return USP_ERR_UNSUPPORTED;
  usp_posdesc qd = {0, Lq, 0, 0};
  usp_posdesc kd[USP_MAX_RING_BLOCKS];
  int acc[USP_MAX_RING_BLOCKS];
  if (causal && (!qpos || !kpos_blocks)) return USP_ERR_NULL;
  if (causal && !desc_ok(qpos, Lq)) return USP_ERR_SHAPE;
  if (causal) qd = *qpos;
  for (int j = 0; j < n_blocks; ++j) {
    if (!k_blocks[j] || !v_blocks[j] || !dk_blocks[j] || !dv_blocks[j]) return USP_ERR_NULL;
    kd[j] = usp_posdesc{0, Lk, 0, 0};
    if (causal) {
      if (!desc_ok(&kpos_blocks[j], Lk)) return USP_ERR_SHAPE;
      kd[j] = kpos_blocks[j];
    }
    acc[j] = accumulate_dkdv[j] ? 1 : 0;
  }
  if (scale == 0.0f) scale = 1.0f / sqrtf((float)hs);
  return launch_ring_attn_bwd(q, k_blocks, v_blocks, kd, n_blocks, d_o, lse, delta, dq, dk_blocks, dv_blocks, bs, Lq,
                              Lk, hq, hkv, hs, scale, causal ? 1 : 0, qd, accumulate_dq ? 1 : 0, acc,
                              (hipStream_t)stream);
} catch (...) {
  return USP_ERR_LAUNCH;
}

namespace {

// Copies of the outputs that usp_ring_attn_bwd_ws keeps in its workspace: dq when its items are cut, every block's
// dk and dv when they have more than one writer per element.
struct RingBwdWs {
  BwdCopies copies;
  int dkdv_copies;
  size_t dq_bytes, kv_bytes_per_block, total;   // dq_bytes / kv_bytes_per_block are 0 where the output is written directly
  size_t ds_bytes, total_with_ds;               // room for dS behind the copies: used when the workspace reaches that far
};

RingBwdWs plan_ring_bwd_ws(int bs, int64_t Lq, int64_t Lk, int hq, int hkv, int hs, int n_blocks) {
  RingBwdWs w;
  w.copies.cut = plan_bwd_cut(bs, Lq, Lk, hq, hkv, n_blocks, true, false);
  w.copies.dq_stride = (size_t)bs * Lq * hq * hs;
  w.copies.dkdv_stride = (size_t)bs * Lk * hkv * hs;
  w.dkdv_copies = (hq / hkv) / w.copies.cut.heads_per_wg * w.copies.cut.q_splits;
  w.dq_bytes = w.copies.cut.k_splits > 1 ? up256(w.copies.dq_stride * sizeof(float) * w.copies.cut.k_splits) : 0;
  w.kv_bytes_per_block = w.dkdv_copies > 1 ? up256(w.copies.dkdv_stride * sizeof(float) * w.dkdv_copies) : 0;
  w.total = w.dq_bytes + 2 * w.kv_bytes_per_block * n_blocks;
  w.ds_bytes = bwd_keeps_ds(hs) ? up256(bwd_ds_bytes(bs, Lq, Lk, hq, n_blocks)) : 0;
  w.total_with_ds = w.total + w.ds_bytes;
  return w;
}

}  // namespace

extern "C" size_t usp_ring_attn_bwd_workspace_bytes(int bs, int64_t Lq, int64_t Lk, int hq, int hkv, int hs,
                                                    int n_blocks) {
  if (bs < 1 || Lq < 1 || Lk < 1 || hq < 1 || hkv < 1 || hq % hkv || (hs != 64 && hs != 128)) return 0;
  if (n_blocks < 1 || n_blocks > USP_MAX_RING_BLOCKS) return 0;
  return plan_ring_bwd_ws(bs, Lq, Lk, hq, hkv, hs, n_blocks).total;
}

extern "C" size_t usp_ring_attn_bwd_workspace_bytes_with_ds(int bs, int64_t Lq, int64_t Lk, int hq, int hkv, int hs,
                                                            int n_blocks) {
  if (bs < 1 || Lq < 1 || Lk < 1 || hq < 1 || hkv < 1 || hq % hkv || (hs != 64 && hs != 128)) return 0;
  if (n_blocks < 1 || n_blocks > USP_MAX_RING_BLOCKS) return 0;
  return plan_ring_bwd_ws(bs, Lq, Lk, hq, hkv, hs, n_blocks).total_with_ds;
}

extern "C" int usp_ring_attn_bwd_ws(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                                    const usp_posdesc* kpos_blocks, int n_blocks, const void* d_o, const float* lse,
                                    const float* delta, float* dq, float* const* dk_blocks, float* const* dv_blocks,
                                    int bs, int64_t Lq, int64_t Lk, int hq, int hkv, int hs, float scale, int causal,
                                    const usp_posdesc* qpos, int accumulate_dq, const int* accumulate_dkdv,
                                    void* workspace, size_t workspace_bytes, void* stream_) try {
  if (!q || !k_blocks || !v_blocks || !d_o || !lse || !delta || !dq || !dk_blocks || !dv_blocks || !accumulate_dkdv)
    return USP_ERR_NULL;
  if (n_blocks < 1 || n_blocks > USP_MAX_RING_BLOCKS) return USP_ERR_UNSUPPORTED;
  if (bs < 1 || Lq < 1 || Lk < 1 || hq < 1 || hkv < 1) return USP_ERR_SHAPE;
  if (hq % hkv) return USP_ERR_DEGREE;
  if (hs != 64 && hs != 128) return USP_ERR_UNSUPPORTED;
  if (!(scale >= 0.0f) || isinf(scale)) return USP_ERR_UNSUPPORTED;
  if (Lq >= (int64_t)1 << 31 || Lk >= (int64_t)1 << 31) return USP_ERR_UNSUPPORTED;
  RingBwdWs w = plan_ring_bwd_ws(bs, Lq, Lk, hq, hkv, hs, n_blocks);
  if (w.total > 0 && (!workspace || workspace_bytes < w.total || ((uintptr_t)workspace & 255))) return USP_ERR_WORKSPACE;
  if (w.ds_bytes && workspace && workspace_bytes >= w.total_with_ds && !((uintptr_t)workspace & 255))
    w.copies.ds = (char*)workspace + w.total;   // room to keep dS between the two kernels
  usp_posdesc qd = {0, Lq, 0, 0};
  usp_posdesc kd[USP_MAX_RING_BLOCKS];
  if (causal && (!qpos || !kpos_blocks)) return USP_ERR_NULL;
  if (causal && !desc_ok(qpos, Lq)) return USP_ERR_SHAPE;
  if (causal) qd = *qpos;
  hipStream_t stream = (hipStream_t)stream_;
  char* ws = (char*)workspace;
  // where the kernels write: the copies in the workspace (always overwritten there), or the outputs themselves
  float* dq_dst = w.dq_bytes ? (float*)ws : dq;
  float* dk_dst[USP_MAX_RING_BLOCKS];
  float* dv_dst[USP_MAX_RING_BLOCKS];
  int acc[USP_MAX_RING_BLOCKS];
  for (int j = 0; j < n_blocks; ++j) {
    if (!k_blocks[j] || !v_blocks[j] || !dk_blocks[j] || !dv_blocks[j]) return USP_ERR_NULL;
    kd[j] = usp_posdesc{0, Lk, 0, 0};
    if (causal) {
      if (!desc_ok(&kpos_blocks[j], Lk)) return USP_ERR_SHAPE;
      kd[j] = kpos_blocks[j];
    }
    if (w.kv_bytes_per_block) {
      dk_dst[j] = (float*)(ws + w.dq_bytes + (size_t)(2 * j) * w.kv_bytes_per_block);
      dv_dst[j] = (float*)(ws + w.dq_bytes + (size_t)(2 * j + 1) * w.kv_bytes_per_block);
      acc[j] = 0;
    } else {
      dk_dst[j] = dk_blocks[j];
      dv_dst[j] = dv_blocks[j];
      acc[j] = accumulate_dkdv[j] ? 1 : 0;
    }
  }
  if (scale == 0.0f) scale = 1.0f / sqrtf((float)hs);
  int st = launch_ring_attn_bwd(q, k_blocks, v_blocks, kd, n_blocks, d_o, lse, delta, dq_dst, dk_dst, dv_dst, bs, Lq, Lk,
                                hq, hkv, hs, scale, causal ? 1 : 0, qd, w.dq_bytes ? 0 : (accumulate_dq ? 1 : 0), acc,
                                stream, &w.copies);
  if (st != USP_OK) return st;
  auto sum_copies = [&](const float* src, float* dst, size_t n, int n_copies, int add) {
    ConvertTensor t;
    t.src = src; t.dst = dst;
    t.n = t.copy_stride = n;
    t.n_copies = n_copies;
    t.add_to_dst = add ? 1 : 0;
    return t;
  };
  if (w.dq_bytes) {
    const ConvertTensor t = sum_copies(dq_dst, dq, w.copies.dq_stride, w.copies.cut.k_splits, accumulate_dq);
    st = launch_bwd_convert(&t, 1, USP_FP32, stream);
    if (st != USP_OK) return st;
  }
  if (w.kv_bytes_per_block)
    for (int j = 0; j < n_blocks; ++j) {
      const ConvertTensor t[2] = {sum_copies(dk_dst[j], dk_blocks[j], w.copies.dkdv_stride, w.dkdv_copies, accumulate_dkdv[j]),
                                  sum_copies(dv_dst[j], dv_blocks[j], w.copies.dkdv_stride, w.dkdv_copies, accumulate_dkdv[j])};
      st = launch_bwd_convert(t, 2, USP_FP32, stream);
      if (st != USP_OK) return st;
    }
  return USP_OK;
} catch (...) {
  return USP_ERR_LAUNCH;
}
