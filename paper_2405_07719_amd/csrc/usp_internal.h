// Internal declarations shared by the translation units of libusp.so (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "usp.h"

namespace usp {

// CUs of the chip the work-splitting plans are made for (MI355X).  The plans (key splits of the forward, slices and
// head splits of the backward) size workspaces, and the workspace queries must work without a GPU, so this is a
// constant and the ONE place it is written; the launchers ask the device for its CU count only to size their grids
// (a plan made for another CU count is still correct, only less well balanced).
constexpr int kPlanCUs = 256;

inline size_t dtype_size(int dt) { return dt == USP_BF16 ? 2 : (dt == USP_FP32 ? 4 : 0); }

// Global position of local index i under a two-run descriptor.
__host__ __device__ inline int64_t pos_of(const usp_posdesc& d, int64_t i) {
  return i < d.len0 ? d.start0 + i : d.start1 + (i - d.len0);
}

// Smallest / largest global position over local indices [a, b), b > a, within the descriptor.
__host__ __device__ inline int64_t pos_min(const usp_posdesc& d, int64_t a, int64_t b) {
  int64_t m = INT64_MAX;
  if (a < d.len0) m = d.start0 + a;
  if (b > d.len0) {
    int64_t a1 = (a > d.len0 ? a : d.len0) - d.len0;
    int64_t v = d.start1 + a1;
    m = v < m ? v : m;
  }
  return m;
}
__host__ __device__ inline int64_t pos_max(const usp_posdesc& d, int64_t a, int64_t b) {
  int64_t m = INT64_MIN;
  if (a < d.len0) {
    int64_t e = b < d.len0 ? b : d.len0;
    m = d.start0 + e - 1;
  }
  if (b > d.len0) {
    int64_t v = d.start1 + (b - 1 - d.len0);
    m = v > m ? v : m;
  }
  return m;
}

// The 256-row tiles that local rows (or keys) [0, len) with positions d are cut into.  Rows of two separate runs under a
// causal mask (the zigzag split of two and more ring ranks): no tile holds rows of both, because it would walk everything
// that the later run sees for the rows of the earlier one as well, one more long item per head.  Measured, ring rank 1 of
// 8, two of L = 16000, 32 heads: eight tiles of 256 in a row, five of them long, 1054 us; four per run 546 us.  Where that
// takes one tile more, as many tiles are long as before: measured in a row / apart, rank 0 of 2 (16 heads) with runs of 808,
// 1064, 1832 rows forward 80.5 / 72.7, 100 / 89.5, 172 / 159 us, backward 153 / 151, 230 / 231, 487 / 472; rank 3 of 8 (32
// heads), 552, 1064, 1832 rows, forward 174 / 176, 434 / 447, 966 / 979, backward 390 / 401, 1130 / 1129, 3154 / 3000.  So
// from eight tiles on, where it gains more than it costs.
struct RowTiles {
  int n, in_run0;     // tiles in all; in_run0 > 0: the first run's, the rest are cut from row len0 on; 0: [0, len) in a row
  int64_t len0, len;
  RowTiles(const usp_posdesc& d, int64_t len_, int causal) : len0(d.len0), len(len_) {
    const bool apart = causal && d.len0 > 0 && d.len1 > 0 && d.start1 != d.start0 + d.len0 && d.len0 % 256 != 0;
    n = (int)((len + 255) / 256);
    in_run0 = 0;
    const int first = (int)((len0 + 255) / 256), both = first + (int)((len - len0 + 255) / 256);
    if (apart && (both == n || n >= 8)) {
      in_run0 = first;
      n = both;
    }
  }
  int64_t begin(int64_t i) const { return in_run0 && i >= in_run0 ? len0 + (i - in_run0) * 256 : i * 256; }
  int64_t end(int64_t i) const {
    const int64_t stop = in_run0 && i < in_run0 ? len0 : len, e = begin(i) + 256;
    return e < stop ? e : stop;
  }
};

// The tiles of n blocks of len rows (keys) each in one backward launch, which cuts all of them in the same places: those of
// RowTiles where it cuts every block alike, else in a row.  (In a whole zigzag ring the last ring rank's two runs adjoin,
// and RowTiles has them in a row: blocks are cut apart for one block at a time, the rows of one rank among them.)
inline RowTiles common_row_tiles(const usp_posdesc* d, int n, int64_t len, int causal) {
  const RowTiles first(d[0], len, causal);
  for (int j = 1; j < n; ++j) {
    const RowTiles x(d[j], len, causal);
    if (x.in_run0 != first.in_run0 || (first.in_run0 && x.len0 != first.len0)) return RowTiles(d[0], len, 0);
  }
  return first;
}

// Places in a forward item's walk over key tiles of KT keys that a wave need not mask: [0, a) and [b0, b1).  They are full tiles
// that lie wholly in one ascending run of the key positions and whose last key no row of the wave precedes (qmin: the first of
// its rows' positions), and so a run of places at the start of each visible range: tiles 0 .. na - 1, then t0 .. t1 - 1.
// A wave without rows (of a query tile that ends with the block or with a run) need not mask any full tile; `all_for_none`: in
// either range, else in the first.  Masked, a tile takes such a wave 3.2 us where its neighbours need 1.8, and the workgroup
// waits for it: 54 tiles of a second run 172 us, without masks 104, and of a cut forward that one item was the time: one of two
// Ulysses ranks of L = 6976, 16 heads, 184 -> 126 us, of L = 5688 128 -> 97; U 8, L = 25008 707 -> 594.  In uncut forwards its
// share is smaller, and the main loops that the compiler then makes are slower: L = 212992 0.3 to 0.5 %.
struct UnmaskedTiles { int a, b0, b1; };
__host__ __device__ inline UnmaskedTiles unmasked_key_tiles(int KT, int causal, bool has_rows, bool all_for_none, int qmin, int start0, int len0,
                                                            int start1, int len1, int Lk, int na, int t0, int t1) {
  const int full = Lk / KT;
  int fa = full, tb0 = 0, tb1 = all_for_none ? full : 0;
  if (causal && has_rows) {
    int64_t c0 = (int64_t)qmin - start0 + 1; c0 = c0 < 0 ? 0 : (c0 > len0 ? len0 : c0);
    int64_t c1 = (int64_t)qmin - start1 + 1; c1 = c1 < 0 ? 0 : (c1 > len1 ? len1 : c1);
    fa = (int)(c0 / KT);
    tb0 = (int)(((int64_t)len0 + KT - 1) / KT);
    tb1 = (int)(((int64_t)len0 + c1) / KT);
  }
  fa = fa < full ? fa : full;
  tb1 = tb1 < full ? tb1 : full;
  return UnmaskedTiles{fa < na ? fa : na, na + (tb0 > t0 ? tb0 : t0) - t0, na + (tb1 < t1 ? tb1 : t1) - t0};
}

// Workgroups of so many threads that one dimension of a grid holds: HIP refuses 2^32 threads and more.
constexpr int64_t max_workgroups(int threads) { return (((int64_t)1 << 32) - 1) / threads; }

inline int launch_status() { return hipGetLastError() == hipSuccess ? USP_OK : USP_ERR_LAUNCH; }

// Raises a kernel's limit of dynamic LDS, once per kernel instance and device (the attribute belongs to the device's
// copy of the function).  `done` is the instance's own record, a function-local static of the caller; later calls,
// which may come during stream capture, only read it.  Two threads that meet here both set the same value.
struct LdsLimitRaised { std::atomic<bool> on_device[64]; };
inline bool raise_dynamic_lds_limit(const void* kernel, size_t bytes, LdsLimitRaised& done) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
  if (done.on_device[dev].load(std::memory_order_acquire)) return true;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
  done.on_device[dev].store(true, std::memory_order_release);
  return true;
}

// Kernel launchers (defined next to their kernels).  All take validated arguments.
// Ranks rank_begin, rank_begin + rank_step, ... below rank_end are transformed in one launch.
// head_rank_base >= 0: the rank whose slot the head-layout base pointer points at (0 for a whole buffer);
// head_rank_base < 0: the head-layout side is a packed workspace holding the launch's ranks back to back.
int launch_layout_a2a(const usp_problem& p, int heads, int dir, const void* src, void* dst, int rank_begin,
                      int rank_end, int head_rank_base, hipStream_t stream, int rank_step = 1);
// The same for up to USP_LAYOUT_MAX_TENSORS tensors of one geometry (same heads, ranks and head_rank_base) in ONE launch.
#define USP_LAYOUT_MAX_TENSORS 3
int launch_layout_a2a_multi(const usp_problem& p, int heads, int dir, int n_tensors, const void* const* src,
                            void* const* dst, int rank_begin, int rank_end, int head_rank_base, hipStream_t stream,
                            int rank_step = 1);
// Optional: Q is read from and O written to the sequence-layout shards of the rank's Ulysses group
// ([U][bs][rows_per_shard][heads][hs], q and o pointing at the group's first shard) instead of dense head-layout
// tensors; head0 is the rank's first head.  Attention kernels: bf16 instance only.  Merge: fp32 partials only (the
// merged O goes to the shards, the merged LSE stays [bs,hq,Lq]).
// kv_heads > 0 (attention forward, batch of one): row-major K and V, too, lie in the shards, rows of kv_heads heads, the
// pointers at the rank's first KV head; 0: dense.
struct SeqLayoutIO { int rows_per_shard, heads, head0, kv_heads = 0; };
// row0 > 0: only the rows [row0, Lq) of every batch are merged (and written); the tensors keep their full shapes.
// part_row0 (with seq): part j holds, of every batch entry, the rows from part_row0[j] on, the first part all that are merged.
int launch_lse_merge(const void* const* o_parts, const float* const* lse_parts, int n_parts, void* o_out,
                     float* lse_out, int bs, int64_t Lq, int hq, int hs, int part_dtype, int out_dtype,
                     hipStream_t stream, const SeqLayoutIO* seq = nullptr, int64_t row0 = 0, const int64_t* part_row0 = nullptr);
// Optional: the running online-softmax state of a ring that delivers its blocks one call at a time (bf16 instance):
// attn_fwd_state_bytes() bytes in the kernel's own layout; first: the state is not read (the call starts it);
// last: the state is not written, the call writes the normalised O and the LSE instead.
struct RingState { float* state; int first, last; };
size_t attn_fwd_state_bytes(int bs, int64_t Lq, int hq, int hs);
int launch_ring_attn_fwd(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                         const usp_posdesc* kpos_blocks, int n_blocks, void* o, float* lse, int bs, int64_t Lq,
                         int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc& qpos,
                         int in_dtype, int o_dtype, hipStream_t stream, const SeqLayoutIO* seq = nullptr,
                         const RingState* state = nullptr, bool v_transposed = false);
// The key-tile-transposed layout of V blocks (USP_SEQ_TO_HEAD_VT): bytes of one rank's block, and the launch that
// writes it for ranks rank_begin, rank_begin + rank_step, ... (packed back to back at dst when head_rank_base < 0,
// else indexed by rank - head_rank_base), straight from the sequence-layout shards.  bf16 data only.
inline size_t vt_block_bytes(int bs, int64_t Lk, int hkv, int hs) {
  return (size_t)bs * hkv * (size_t)((Lk + 63) / 64) * 64 * hs * 2;
}
int launch_layout_a2a_vt(const usp_problem& p, int heads, const void* src, void* dst, int rank_begin, int rank_end,
                         int head_rank_base, hipStream_t stream, int rank_step = 1);
// Key split: the same query rows against n_blocks blocks, every (query tile, head, batch, block) its own work item of
// ONE launch, each block's result (fp32 O, LSE) in its own partial, to be merged by launch_lse_merge.  Block j holds
// lk_blocks[j] <= Lk keys (all Lk when lk_blocks is null); Lk is the batch stride, in rows, of every block's tensors.
// With `mixed`, only the LAST n_split_tiles query tiles of the block (first in item order, the heaviest under a causal
// mask) are cut so; the other query tiles are whole items of the same launch that walk
// all blocks and write their finished rows (bf16, through `seq` when given) to mixed->o and mixed->lse.  The partials
// then hold the rows of the cut tiles only, to be merged over that row range.
// v_transposed: the V pointers are pieces of blocks in key-tile-transposed layout (each begins at a tile of 64 keys of
// its block; Lk, the batch stride in rows, then also gives the number of tiles per head of a whole block).
// listed, n_listed: the launch's items (listed_item(), at most kMaxListedItems), heaviest first, each to run for every head
// and batch entry; pieces that a tile sees nothing of are not among them.  Without a list every one of the last
// n_split_tiles tiles has an item per piece.  part_row0: the first row that the piece's partial result holds (null: 0).
struct MixedLaunch {
  void* o;
  float* lse;
  int n_split_tiles;
  bool v_transposed;
  const uint16_t* listed = nullptr;
  int n_listed = 0;
  const int64_t* part_row0 = nullptr;
};
constexpr int kMaxListedItems = 1024, kListedTileBits = 11, kListedWhole = 31;
constexpr uint16_t listed_item(int tile, int piece) { return (uint16_t)(piece << kListedTileBits | tile); }   // piece kListedWhole: all of them
static_assert(kMaxListedItems <= 1 << kListedTileBits && USP_MAX_RING_BLOCKS < kListedWhole, "every tile and piece has a number");
int launch_attn_fwd_partials(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                             const usp_posdesc* kpos_blocks, const int* lk_blocks, int n_blocks, float* const* o_parts,
                             float* const* lse_parts, int bs, int64_t Lq, int64_t Lk, int hq, int hkv, int hs,
                             float scale, int causal, const usp_posdesc& qpos, hipStream_t stream,
                             const SeqLayoutIO* seq = nullptr, const MixedLaunch* mixed = nullptr);
int launch_block_attn_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int bs, int64_t Lq,
                          int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc& qpos,
                          const usp_posdesc& kpos, int in_dtype, int o_dtype, hipStream_t stream, const RingState* state = nullptr);

// wave_split_attn_fwd.hip: the keys of 32 query rows split over the waves of one workgroup; bf16 or fp32 data.
// The whole of Algorithm 1's forward for ranks [rank_begin, rank_end) in one launch, everything read and written in the
// sequence-layout shards, no workspace; and one ring step on dense tensors.
int launch_wave_split_usp_fwd(const usp_problem& p, const void* q, const void* k, const void* v, void* o, float* lse,
                              int rank_begin, int rank_end, float scale, hipStream_t stream);
int launch_wave_split_block_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int bs, int64_t Lq,
                                int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc& qpos,
                                const usp_posdesc& kpos, int in_dtype, int o_dtype, hipStream_t stream,
                                const RingState* state = nullptr);
// Time of such a launch, in us: rounds of one workgroup (32 rows of a head; two at head size 64) per CU, 4 us each for its
// first loads and the merge of its waves, and 0.6 PFLOP/s, where reading every key for only 32 rows leaves it.  Measured
// (this formula): one rank of four heads, causal, L = 4096 34 us (41), 8192 116 (134); 32 heads, L = 1024 31 (34),
// 2048 80 (93); four heads of size 64, L = 4096 22 (22), 6144 40 (44).
inline double wave_split_us(int64_t rows, int heads, int hs, double flop) {
  const int64_t wgs = (rows + 31) / 32 * heads, round = hs == 64 ? 2 * kPlanCUs : kPlanCUs;
  return 4.0 + 4.0 * (double)((wgs + round - 1) / round) + flop / 0.6e9;
}

// Where one block of keys goes, to the waves of a workgroup or to 256-row items.
// fp32 has the one kernel.  bf16: the launch of 256-row items takes 6 us and its longest item (1.75 us per 64 keys at
// head size 128), or its work at 1.1 (0.8) PFLOP/s; short blocks, whose items are few and long, are faster with their
// keys split over the waves of a workgroup.  Measured, the ring of 32/8 heads, one call per block and the merge, 256-row
// items against waves: 8 blocks of 256 keys 145 / 74 us, of 512 keys 178 / 126, 2 blocks of 1024 keys 78 / 83; head size
// 64: 8 blocks of 512 keys 132 / 73, 2 of 1024 56 / 56.  With the running state (either kernel reads and writes the
// same records): 16 heads, 8 blocks of 452 keys 200 / 78, of 1024 keys 233 / 143; head size 64: 164 / 70, 170 / 78.
inline bool block_goes_to_waves(int bs, int64_t Lq, int64_t Lk, int hq, int hs, int causal, int dtype) {
  const double flop = 4.0 * hs * bs * hq * (double)Lq * (double)Lk * (causal ? 0.5 : 1.0);
  return dtype == USP_FP32 || wave_split_us(Lq, bs * hq, hs, flop) <
                                  6.0 + std::max(1.75 * (double)Lk / 64 * (hs / 128.0), flop / (hs == 128 ? 1.1e9 : 0.8e9));
}

// Whether the second product runs a tile behind (block_attn_fwd.hip, TRAILING; head size 64): blocks of Lk keys, of which an item
// walks `piece` at a time on the average (Lk, where the keys are not cut).  Every block or piece fills and drains a pipeline that is a tile longer, with
// steps that copy scores and weights.  Without / with it, one rank, us.  Blocks: ring 4, 962 keys 75.4 / 79.5, ring 8, 1502 123.8 / 131.4,
// ring 4, 1646 99.9 / 101.5, steps with a state, 834 86.3 / 88.5, steps with partial results, 1764 143.4 / 146.5; on the other side
// 1292 100.8 / 99.4, 1852 187.2 / 185.7, 1928 117.5 / 113.2, 4096 611 / 593.  (An even number of tiles is drained in four such steps, an odd one in
// three.)  Pieces of blocks that are long enough, most of them without a mask: 888 keys 111.0 / 112.1, 1156 51.1 / 51.8, 1223 129.0 / 132.5,
// 1270 193.3 / 191.7, 1522 201.5 / 198.9, 1558 212.2 / 205.4, 1751 143.1 / 140.5, 1928 69.0 / 70.1, 2138 210.1 / 206.3; of 23 from 1270 to 2666 keys
// three lose, 1.6 and 5 % where two pieces under a mask are all that a CU has (L = 4960 85.6 / 89.9).
inline bool second_product_trails(int64_t Lk, int64_t piece) { return Lk >= 2048 && piece >= 1250; }

// Rows per workgroup of an fp32 launch: 16 where workgroups of 32 leave half of the CUs idle, or, under a causal mask, hold them
// with items of very different lengths: then only with walks of a twelfth as many key tiles as there are workgroups, for twice
// as many of these do not fit the chip at once and each has its own first loads and merge.  Measured, 32 and 16 rows, us (in
// brackets workgroups of 32, and tiles): no mask, four ranks of L = 256 (32) 8.6, 6.5; L = 512, head size 128 (64) 21, 13.5;
// L = 1024, head size 128 (128) 36.6, 22.6; L = 2048, head size 128 (256) 68.7, 75.7; causal, head size 64, L = 128 (144, 4) 7.3,
// 9.4, L = 256 (256, 8) 9.4, 10.9, four ring ranks (144, 8) 9.8, 11.3; L = 384 (144, 12) 10.9, 9.3, (252, 12) 11.2, 12.8; L = 512
// (192, 16) 13.1, 11.5, (256, 16) 13.1, 12.7, with four ring ranks 13.5, 15.0; L = 768 (240, 24) 17.3, 15.0, with four 17.95, 17.96;
// L = 1024 (256, 32) 21.3, 17.2; head size 128 the same within 0.1 of the ratio; L = 2048 (512, 64) 43.0, 50.0.
inline int wave_split_fp32_rows(int64_t Lq, int64_t heads, int64_t key_tiles, int causal) {
  const int64_t wgs = (Lq + 31) / 32 * heads;
  return wgs <= kPlanCUs / 2 || (causal && wgs <= kPlanCUs && wgs <= 12 * key_tiles) ? 16 : 32;
}

// Whether tiles cross from one shard of n rows into the next.  By shards there are more of them, and emptier ones: with eight
// shards of 34 rows 16 for 9.  They cross where that makes up for the rows' offsets, counted in rounds of the eight waves and half
// in tiles, for the waves share what loads: at head size 128 and 32 rows per workgroup always, in bf16 at head size 64 with four
// shards and more always and with fewer for a twentieth, else for more.  (In 32 bits: the offset of a tile's last row, jumps included.)  Measured, by shards and crossing, us,
// a batch of two: 32/8 heads, one rank of U 8 x R 4, shards of 34 rows 18.9, 12.4, of 24 rows 12.5, 10.4; U 4 x R 2, 16/8 heads, all
// ranks, shards of 130 43.4, 41.2, of 330 150.6, 148.0; fp32, eight heads, U 8 x R 2, all ranks, shards of 34 72.5, 50.1, of 520
// 4648, 4421; bf16, head size 64, one rank, U 8 x R 2, shards of 100 13.1, 10.5, of 266 30.0, 29.4, U 4 x R 2, contiguous, of 130 10.9,
// 10.2, of 236 16.9, 15.6, U 4, of 130 7.1, 7.4, U 2 x R 2, all ranks, of 66 8.4, 8.7, of 130 13.2, 13.5; fp32, head size 64, U 8 x R 4, all ranks, of 34 116, 73, U 8 x R 2, one rank, of 200 36.2, 35.2, of 266
// 78.3, 80.5; fp32, 16 rows per workgroup, U 2 x R 2, of 34 9.8, 10.1, of 130 47.7, 49.3.
constexpr int kWaveSplitWaves = 8, kWaveSplitTile = 32;
enum Cross { kNoCross, kOneCross, kAnyCross };   // kOneCross: a tile crosses once at most
inline Cross wave_split_crossing(int64_t n, int U, int R, int bs, int64_t row_bytes, int dtype, int hs, int rows) {
  constexpr int T = kWaveSplitTile, W = kWaveSplitWaves;
  if (bs == 1 || U == 1 || n % T == 0 || (T + (n + T) * (bs - 1)) * row_bytes >= (int64_t)1 << 31) return kNoCross;
  auto cost = [](int64_t tiles) { return 2.0 + (double)((tiles + W - 1) / W) + (double)tiles / W; };
  const int64_t by_shard = (int64_t)R * U * ((n + T - 1) / T), crossing = R * ((U * n + T - 1) / T);
  const double offsets = (hs == 128 && rows == 32) || (dtype == USP_BF16 && U >= 4) ? 1.0 : dtype == USP_BF16 ? 1.05 : 1.07;
  if (cost(by_shard) <= offsets * cost(crossing)) return kNoCross;
  return n < T ? kAnyCross : kOneCross;
}

// One tensor of the launch that prepares a backward: rows [r0, r0 + n_rings) x columns [c0, c0 + n_cols) of ring blocks of the
// sequence layout [N][bs][L/U][heads][hs].  dst: their copy in [block][bs][head][row][hs]; o (src is dO): D_i of their rows,
// [block][bs][head][row] fp32 at delta.
struct PrepareTensor {
  const void* src;
  const void* o;
  void* dst;
  float* delta;
  int U, r0, n_rings, c0, n_cols, heads, heads_per_rank;
};
int launch_bwd_prepare(const PrepareTensor* tensors, int n_tensors, int bs, int64_t L, int hs, hipStream_t stream);
// How a backward launch pair divides its work (plan_bwd_cut): query heads of a KV group walked by one dK/dV
// workgroup, slices of a dQ item's key tiles, slices of a dK/dV item's query tiles.
struct BwdCut { int heads_per_wg, k_splits, q_splits; };
// equal_items: no causal mask (usp_attn_bwd knows; the per-call entry points, whose workspace query does not, say false).
BwdCut plan_bwd_cut(int bs, int64_t Lq, int64_t Lk, int hq, int hkv, int n_blocks, bool cut_items, bool equal_items);
// Room for copies of the outputs, one per slice: dq holds cut.k_splits copies dq_stride elements apart, every block's
// dk and dv hold (hq / hkv / cut.heads_per_wg) * cut.q_splits copies dkdv_stride elements apart; every copy is
// written (or added to, as the accumulate flags say) in full, nothing is atomic; launch_bwd_convert adds them up.
// ds (optional, null = off): room for the dS of one launch pair, bwd_ds_bytes() bytes: the dK/dV kernel then runs
// first and writes the dS blocks it forms, and the dQ kernel reads them back instead of forming S and dP again
// (5 matrix products per tile pair instead of 7, for 2 bytes written and read per visible pair).
struct BwdCopies { BwdCut cut; size_t dq_stride, dkdv_stride; void* ds = nullptr; };
// Where a launch pair finds its tensors when that is not dense row-major head layout [bs][L][heads][hs]: row i of head h of
// (block, batch entry) rb lies rb * block + i * row + h * head rows of hs elements into the tensor.
struct RowPlace { int64_t block; int row, head; };
// dq_heads / dkdv_heads > 0: the results leave as bf16, in rows of that many heads, for outputs with one writer per element
// that nothing is added to.  n_qblk > 1: Q, dO, LSE, delta and dQ hold the rows of that many ring ranks back to back, each
// with its own positions (no kept dS; dq_heads > 0).
struct BwdPlace {
  RowPlace q, kv;
  int dq_heads, dkdv_heads;
  int n_qblk;
  const usp_posdesc* qpos_blocks;
};
constexpr bool bwd_keeps_ds(int hs) { return hs >= 128; }   // see plan_bwd
inline size_t bwd_ds_bytes(int bs, int64_t Lq, int64_t Lk, int hq, int n_blocks) {
  return (size_t)bs * hq * n_blocks * (size_t)((Lk + 255) / 256 * 8) * (size_t)((Lq + 255) / 256 * 8) * 2048;
}
int launch_ring_attn_bwd(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                         const usp_posdesc* kpos_blocks, int n_blocks, const void* d_o, const float* lse,
                         const float* delta, float* dq, float* const* dk_blocks, float* const* dv_blocks, int bs,
                         int64_t Lq, int64_t Lk, int hq, int hkv, int hs, float scale, int causal,
                         const usp_posdesc& qpos, int accumulate_dq, const int* accumulate_dkdv, hipStream_t stream,
                         const struct BwdCopies* copies = nullptr, const struct BwdPlace* io = nullptr);
int launch_block_attn_bwd(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                          const float* delta, float* dq, float* dk, float* dv, int bs, int64_t Lq, int64_t Lk, int hq,
                          int hkv, int hs, float scale, int causal, const usp_posdesc& qpos, const usp_posdesc& kpos,
                          int accumulate_dq, int accumulate_dkdv, hipStream_t stream);
// One tensor of a conversion: dst[i] = sum over n_copies of src[c * copy_stride + i], i < n, for n_blocks blocks src_blk and
// dst_blk elements apart, converted (fp32 output: optionally added to dst).  seq: the result goes to the sequence-layout
// shards of the rank's Ulysses group (dst = the group's first shard) instead of the dense [bs, rows, heads, hs] tensor the
// source is: the reverse all-to-all of Algorithm 1 rides on the conversion's stores.
struct ConvertTensor {
  const float* src;
  void* dst;
  size_t n, copy_stride;
  int n_copies;
  int add_to_dst = 0;
  int n_blocks = 1;
  size_t src_blk = 0, dst_blk = 0;
  uint64_t absent = 0;   // bit b: block b (of at most 64) has no source, zeros are written
  const SeqLayoutIO* seq = nullptr;
  int bs = 0;
  int64_t rows = 0;
  int heads = 0, hs = 0;
};
// Up to three of them in one launch.
int launch_bwd_convert(const ConvertTensor* tensors, int n_tensors, int out_dtype, hipStream_t stream);

}  // namespace usp
