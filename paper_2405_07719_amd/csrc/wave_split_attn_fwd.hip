// Attention forward with the keys of 32 query rows split over the eight waves of ONE workgroup: the whole ring loop of
// Algorithm 1 (all-to-alls, blocks, merge) for a range of virtual ranks in a single launch, for the problems where
// launches and latency are the time rather than the matrix core, and for fp32 data of every size.
//
//   * A workgroup owns 32 query rows of one (rank, batch, head).  Its waves take the visible 32-key tiles of all K/V
//     blocks in turn (tile j of the walk to wave j mod 8), each with an online-softmax state of its own, and combine the
//     eight states through LDS at the end: the key split and its merge cost two barriers instead of fp32 partials in
//     memory and a launch.  A rank of 512 rows is 16 workgroups per head here where the 256-row kernel has 2.
//   * Q, K and V are read and O is written where the caller holds them, in the sequence-layout shards: the all-to-alls
//     are address arithmetic.  (Consecutive shards of one batch entry are contiguous when bs = 1.)
//   * Ranks, batch and heads are the grid: all ranks of a range run side by side.
//   * Operands.  Waves share no keys: each passes its K tile through a tile of LDS of its own (whole rows in, fragments
//     out: A operand of S^T = K Q^T, lane = key).  bf16: V rows follow through the same tile and come back by transpose
//     reads.  fp32: v_mfma_f32_32x32x2_f32 takes ONE value per lane and product, so V needs no transposition at all:
//     product i multiplies the two keys that the lane halves hold in score register i with 32 head dims, lane = dim.
// What bounds it.  Small problems: the chain of latencies of one workgroup (arguments, Q, K and V, two products, merge,
// store: 6 us), so the prologue has no divisions, the merge no dependent LDS reads, a tile's loads no branches (loops over
// the waves with a run-time bound alone cost 15 %: eight LDS reads, each waited for).  Large ones: every workgroup reads
// all its keys for only 32 rows, eight times the L2 and LDS traffic per product of the 256-row kernel: 0.54 PFLOP/s at
// L = 8192, where that one has 0.71 (K fragments loaded straight from their rows, 32 lines per instruction, had 0.39).
// Where the line between the two lies is in usp_api.cpp (short_in_one_launch).  fp32: the matrix core at fp32 rate, 124
// TFLOP/s at L = 2048, eight heads of size 128, no mask (154 is what a large fp32 matrix product reaches); one thread per row on the vector
// ALU, as it was before, took 1230 us for the four ranks of L = 256 that take 9 us here, and the four bf16 ranks of
// L = 1024 took 121 us in nine launches where this is one of 12 us.
#include <algorithm>

#include "attn_device.h"
#include "usp_internal.h"

namespace usp {
namespace {

using namespace dev;

constexpr int kWaves = 8, kRows = 32, kTile = 32;

// The caller's tensors lie on an element's alignment, no more is claimed (this chip's wide accesses take any address).
typedef bf16x8 bf16x8_any __attribute__((aligned(2)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));

struct WsArgs {
  const void* q;
  const void* k;
  const void* v;
  void* o;
  float* lse;
  int bs, hq, hkv, g;         // heads of one rank
  int q_heads, kv_heads;      // heads in a row of Q / O and of K / V
  int U, R, rank_begin, n_ranks;
  int first_wg;               // work items before this launch's first (0 but for 2^32 threads and more; a second grid
                              // dimension instead: 12.37 us for 12.17)
  FastDiv n_q, n_k;           // rows of a Q and of a K/V shard
  FastDiv by_hkv, by_bs, by_ranks, by_g, by_U;
  int Lq, Lk;                 // rows of a ring block
  int n_qtiles, causal, split;
  PosDesc32 qpos, kpos;       // split < 0: the one block's positions as given, else by Algorithm 2 from the ring rank
  float scale, scale_log2;
  // Running state of a ring that delivers its blocks one per call (STATE instances), in the 256-row kernel's records
  // (block_attn_fwd.hip): per 32 rows of a (batch, head) the O^T accumulator as [hs / 8][64 lanes][4], m, and l, per lane.
  float* state;
  int state_first, state_last, state_records;   // records of a (batch, head)
};

// Algorithm 2 for ring rank r: chunks r and 2R-1-r of 2R, or block r of R
__device__ inline PosDesc32 block_positions(const WsArgs& a, const PosDesc32& given, int len, int r) {
  if (a.split < 0) return given;
  if (a.split == USP_SPLIT_ZIGZAG) {
    const int c = len / 2;
    return PosDesc32{r * c, c, (2 * a.R - 1 - r) * c, c};
  }
  return PosDesc32{r * len, len, 0, 0};
}

// The rows of a ring block (one batch entry, one head) inside the shards [U][bs][n][heads][hs]: row j lies at
// base + j row_bytes + (j / n) jump, and jump is 0 when bs = 1.
struct BlockRows {
  const char* base;
  FastDiv n;
  uint32_t row_bytes;
  int64_t jump;
  __device__ const char* row(int j) const { return base + (int64_t)j * row_bytes + (int64_t)n.div(j) * jump; }
};

__device__ inline BlockRows block_rows(const void* t, int esize, int hs, int bs, FastDiv n, int heads, int first_shard, int b, int head) {
  const uint32_t row_bytes = (uint32_t)heads * hs * esize;
  const int64_t run_bytes = (int64_t)n.d * row_bytes, shard_bytes = bs * run_bytes;
  return BlockRows{(const char*)t + first_shard * shard_bytes + b * run_bytes + (int64_t)head * hs * esize, n, row_bytes,
                   shard_bytes - run_bytes};
}

// One 32-key tile of such rows.  Inside one shard (always, when bs = 1) it is read through a buffer descriptor whose extent
// ends with the last valid row: rows past it read as zeros.  The row within the tile is part of the vector offset, which
// the descriptor's range check covers (the scalar offset it does not).  Row addresses of 64 bits took as long as the products
// (and cost the ragged last tile 1 to 3 us at L = 250 to 2000: fp32, head size 64, L = 248 10.8 us for 10.0).  A tile that
// crosses from one shard into the next, which lie bs entries apart, finds each row on its own, clamped to the last.
// kScalarStep: the row goes into the scalar offset instead, and a ragged tile, too, finds its rows on its own (bf16 at head
// size 64, whose 128 registers hold no offset per load: L = 1024 18.25 us, with the vector offset 19.1).
template <bool kScalarStep>
struct Tile {
  BlockRows rows;
  int key0, last;       // first key; last valid row of the tile
  bool whole;           // read through the descriptor
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ Tile(const BlockRows& r, int key0_, int len, int row_len) : rows(r), key0(key0_) {
    last = min(kTile, len - key0) - 1;
    whole = (!kScalarStep || last == kTile - 1) && (r.jump == 0 || r.n.div(key0) == r.n.div(key0 + last));
    rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)r.row(key0), 0, last * (int)r.row_bytes + row_len, kRawBufferFlags);
  }
  // t[i] = 16 bytes (8: V of the fp32 kernel at head size 64) at byte `col` of row lane_row + step(i)
  template <bool kWhole, typename V, int N, typename Step>
  __device__ void load(V (&t)[N], int lane_row, Step step, int col) const {
    static_assert(sizeof(V) == 16 || sizeof(V) == 8, "");
    typedef V VAny __attribute__((aligned(2)));
    const int at = lane_row * (int)rows.row_bytes + col;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int row = step(i) * (int)rows.row_bytes, voff = kScalarStep ? at : at + row, soff = kScalarStep ? row : 0;
      if constexpr (!kWhole) t[i] = *(const VAny*)(rows.row(key0 + min(lane_row + step(i), last)) + col);
      else if constexpr (sizeof(V) == 16) t[i] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, soff, 0));
      else t[i] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(rsrc, voff, soff, 0));
    }
  }
};

// ---- operands of one data type: the fragments of Q and of a 32-key tile, and the two products -------------------
template <typename T, int HS> struct Operands;

template <int HS> struct Operands<__bf16, HS> {
  static constexpr int KSTEPS = HS / 16, DB = HS / 32, CPR = HS / 8;
  static constexpr int kWavesPerSimd = HS == 64 ? 4 : 2;   // head size 64: two workgroups to a CU
  // Rows of the wave's LDS tile.  K: an odd number of 16-byte chunks, no bank conflicts on the fragment reads; V: an odd
  // multiple of 64 bytes, none on the transpose reads.  K and V take turns in one tile (a wave's LDS accesses are in order).
  static constexpr int KSTR = HS * 2 + 48, VSTR = HS * 2 + 64;
  static constexpr int kLdsPerWave = kTile * VSTR;
  static constexpr int TL = kTile * CPR / 64;            // 16-byte loads per lane of a tile
  typedef Tile<HS == 64> KvTile;
  bf16x8 q[KSTEPS];
  u32x4 k[TL], v[TL];

  __device__ void load_q(const char* row, int hl) {
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) q[ks] = *(const bf16x8_any*)(row + 32 * ks + 16 * hl);
  }
  template <bool kWhole> __device__ static void load_rows(u32x4 (&t)[TL], const KvTile& tile, int lane) {
    tile.template load<kWhole>(t, lane / CPR, [](int c) { return c * (64 / CPR); }, (lane % CPR) * 16);
  }
  template <int STR> __device__ static void stash_rows(char* lds, const u32x4 (&t)[TL], int lane) {
#pragma unroll
    for (int c = 0; c < TL; ++c) {
      const int ch = lane + 64 * c;
      *(u32x4*)(lds + (ch / CPR) * STR + (ch % CPR) * 16) = t[c];
    }
    __builtin_amdgcn_wave_barrier();   // this wave's own LDS accesses stay in this order
  }
  template <bool kWhole> __device__ void load_tile(const KvTile& kt, const KvTile& vt, int lane) {
    load_rows<kWhole>(k, kt, lane);
    load_rows<kWhole>(v, vt, lane);
  }
  __device__ void stash_k(char* lds, int lane) { stash_rows<KSTR>(lds, k, lane); }
  // S^T = K Q^T; leaves V in the LDS tile
  __device__ f32x16 scores(char* lds, int lane) {
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    const char* row = lds + (lane & 31) * KSTR + 16 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(row + 32 * ks), q[ks], s, 0, 0, 0);
    __builtin_amdgcn_wave_barrier();
    stash_rows<VSTR>(lds, v, lane);
    return s;
  }
  // O^T += V^T P^T; p = the tile's 16 weights of this lane
  __device__ void accumulate(const f32x16& p, f32x16 (&o)[DB], const char* lds, int lane) {
    const int hl = lane >> 5, grp = lane >> 4, j16 = lane & 15;
    const char* vlane = lds + (4 * hl + (j16 >> 2)) * VSTR + (16 * (grp & 1) + 4 * (j16 & 3)) * 2;
    __builtin_amdgcn_wave_barrier();   // the tile was written by this wave's own, in-order LDS stores
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      u32x4 pk;
#pragma unroll
      for (int pr = 0; pr < 4; ++pr) pk[pr] = pack_bf16(p[8 * s + 2 * pr], p[8 * s + 2 * pr + 1]);
      const bf16x8 pf = __builtin_bit_cast(bf16x8, pk);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const char* p0 = vlane + (16 * s) * VSTR + db * 64;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0 + 8 * VSTR));
        const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf, o[db], 0, 0, 0);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  // head dim of element e of register group j (registers 4j .. 4j + 3) of block db: four consecutive dims from here
  static __device__ int dim4(int db, int j, int hl) { return 32 * db + 8 * j + 4 * hl; }
  static __device__ f32x4 out4(const f32x16 (&o)[DB], int db, int j) {
    return f32x4{o[db][4 * j], o[db][4 * j + 1], o[db][4 * j + 2], o[db][4 * j + 3]};
  }
  static constexpr int kGroups = DB * 4;   // groups of four dims per lane
  static __device__ int group_dim(int gi, int hl) { return dim4(gi / 4, gi % 4, hl); }
  static __device__ f32x4 group(const f32x16 (&o)[DB], int gi) { return out4(o, gi / 4, gi % 4); }
};

template <int HS> struct Operands<float, HS> {
  static constexpr int DB = HS / 32, KC = HS / 8, CPR = HS / 4;
  static constexpr int kWavesPerSimd = 2;
  static constexpr int KSTR = HS * 4 + 16;               // an odd number of 16-byte chunks
  static constexpr int kLdsPerWave = kTile * KSTR;
  static constexpr int TL = kTile * CPR / 64;
  typedef Tile<false> KvTile;
  typedef float vrow __attribute__((ext_vector_type(DB)));
  f32x4 q[KC];           // dims 8 c + 4 (lane half) .. + 3: the product's two k indices are the lane halves
  f32x4 k[TL];           // a tile's K rows on their way to LDS
  vrow v[16];            // V of the key that score register i of this lane half holds, dims DB l32 .. + DB - 1

  __device__ void load_q(const char* row, int hl) {
#pragma unroll
    for (int c = 0; c < KC; ++c) q[c] = *(const f32x4_any*)(row + 32 * c + 16 * hl);
  }
  template <bool kWhole> __device__ void load_tile(const KvTile& kt, const KvTile& vt, int lane) {
    kt.template load<kWhole>(k, lane / CPR, [](int c) { return c * (64 / CPR); }, (lane % CPR) * 16);
    if constexpr (HS == 64) load_v<kWhole>(vt, lane);
  }
  template <bool kWhole> __device__ void load_v(const KvTile& vt, int lane) {
    vt.template load<kWhole>(v, 4 * (lane >> 5), [](int i) { return 8 * (i >> 2) + (i & 3); }, (lane & 31) * (DB * 4));
  }
  __device__ void stash_k(char* lds, int lane) {
#pragma unroll
    for (int c = 0; c < TL; ++c) {
      const int ch = lane + 64 * c;
      *(f32x4*)(lds + (ch / CPR) * KSTR + (ch % CPR) * 16) = k[c];
    }
    __builtin_amdgcn_wave_barrier();
  }
  __device__ f32x16 scores(char* lds, int lane) {
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    const char* row = lds + (lane & 31) * KSTR + 16 * (lane >> 5);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const f32x4 kc = *(const f32x4*)(row + 32 * c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float ka = kc[e], qa = q[c][e];
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka, qa, s, 0, 0, 0);
      }
    }
    __builtin_amdgcn_wave_barrier();
    return s;
  }
  __device__ void accumulate(const f32x16& p, f32x16 (&o)[DB], const char*, int) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float pi = p[i];
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const float va = v[i][db];
        o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(va, pi, o[db], 0, 0, 0);
      }
    }
  }
  // register i of block db is head dim DB (row i of the product) + db
  static constexpr int kGroups = DB * 4;
  static __device__ int group_dim(int gi, int hl) {
    const int r = DB == 4 ? gi : 2 * gi;                 // the product rows of this group: one (DB = 4) or two (DB = 2)
    return DB * (8 * (r >> 2) + 4 * hl + (r & 3));
  }
  static __device__ f32x4 group(const f32x16 (&o)[DB], int gi) {
    if constexpr (DB == 4) return f32x4{o[0][gi], o[1][gi], o[2][gi], o[3][gi]};
    else return f32x4{o[0][2 * gi], o[1][2 * gi], o[0][2 * gi + 1], o[1][2 * gi + 1]};
  }
};

template <typename T, int HS>
constexpr size_t lds_bytes() {
  const size_t states = (size_t)kWaves * kRows * (HS + 4) * sizeof(float), tiles = (size_t)kWaves * Operands<T, HS>::kLdsPerWave;
  return (states > tiles ? states : tiles);
}

template <typename T, int HS, typename OutT, bool STATE = false>
__global__ __attribute__((amdgpu_flat_work_group_size(kWaves * 64, kWaves * 64), amdgpu_waves_per_eu(Operands<T, HS>::kWavesPerSimd, Operands<T, HS>::kWavesPerSimd)))
void wave_split_attn_fwd(const WsArgs a) {
  using Op = Operands<T, HS>;
  constexpr int DB = HS / 32, OSTR = HS + 4;   // floats between the rows of a state in LDS: an odd number of 16 B chunks
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ float m_s[kWaves][kRows], l_s[kWaves][kRows], inv_s[kRows], first_s[2][kRows];
  const int lane = threadIdx.x & 63, l32 = lane & 31, hl = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

  // KV group fastest (neighbouring workgroups go to different XCDs: one XCD's L2 then holds few KV heads), then head,
  // then query tile, heaviest first under a causal mask
  int kvh = a.first_wg + (int)blockIdx.x;
  int b = a.by_hkv.split(kvh);
  int rank = a.by_bs.split(b);
  int hg = a.by_ranks.split(rank);
  const int t = a.by_g.split(hg);
  rank += a.rank_begin;
  int u = rank;
  const int r = a.by_U.split(u);
  const int h = kvh * a.g + hg;
  const int row0 = (a.causal ? a.n_qtiles - 1 - t : t) * kRows, row1 = min(a.Lq, row0 + kRows);
  const PosDesc32 qpos = block_positions(a, a.qpos, a.Lq, r);
  const int qmin = a.causal ? pos_min(qpos, row0, row1) : 0;
  const int my_row = min(row0 + l32, a.Lq - 1);
  const int qp = a.causal ? pos_of(qpos, my_row) : 0;

  Op op;
  const BlockRows qr = block_rows(a.q, sizeof(T), HS, a.bs, a.n_q, a.q_heads, r * a.U, b, u * a.hq + h);
  op.load_q(qr.row(my_row), hl);

  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  float m = -INFINITY, l = 0.f;

  // The state enters with the merge, as a ninth wave's would, and leaves from there: nothing of it is held meanwhile.
  float* rec = nullptr;
  __shared__ float m_state_s[kRows], f_state_s[kRows];
  if constexpr (STATE) {
    rec = a.state + ((size_t)(b * a.hq + h) * a.state_records + row0 / kRows) * (HS * kRows + 128);
    if (!a.state_first && !a.state_last) {   // rows that see nothing of this block: their state stays as it is
      const TileRanges tr = visible_key_tiles<kTile>(a.causal, qpos, a.kpos, a.Lk, row0, row1);
      if (tr.a1 - tr.a0 + tr.b1 - tr.b0 == 0) return;   // workgroup-uniform
    }
    if (threadIdx.x < kRows) m_state_s[threadIdx.x] = a.state_first ? -INFINITY : rec[HS * kRows + threadIdx.x];
  }

  char* const lds = smem + wave * Op::kLdsPerWave;
  int turn = wave;        // tiles of the walk until this wave's next one
  // bf16: every wave starts from the row maxima over the walk's first 64 keys, which waves 0 and 1 hold after their first
  // products, and moves on from them only where a row grows by more than 2^8 (P is then bounded by that instead of 1).
  // The weights are rounded to bf16 as in the 256-row kernel that way, to the same bits where its items begin with the same
  // keys, and the O that the two leave a backward differ by the order of fp32 sums instead of by a rounding in every
  // weight.  Costs one barrier (12.2 -> 12.4 us at four ranks of L = 1024).
  constexpr bool kShareFirst = sizeof(T) == 2;
  constexpr float kRescaleThreshold = kShareFirst ? 8.f : 0.f;   // log2 units
  bool shared_first = !kShareFirst;   // wave-uniform: every wave passes the one barrier exactly once
  for (int i = 0; i < a.R; ++i) {
    const int blk = r - i < 0 ? r - i + a.R : r - i;   // Algorithm 1 step 5: step i visits block (r - i) mod R
    const PosDesc32 kpos = block_positions(a, a.kpos, a.Lk, blk);
    const TileRanges tr = visible_key_tiles<kTile>(a.causal, qpos, kpos, a.Lk, row0, row1);
    const int na = tr.a1 - tr.a0, nt = na + (tr.b1 - tr.b0);
    const BlockRows kr = block_rows(a.k, sizeof(T), HS, a.bs, a.n_k, a.kv_heads, blk * a.U, b, u * a.hkv + kvh);
    const BlockRows vr = block_rows(a.v, sizeof(T), HS, a.bs, a.n_k, a.kv_heads, blk * a.U, b, u * a.hkv + kvh);
    for (; turn < nt; turn += kWaves) {
      const int key0 = (turn < na ? tr.a0 + turn : tr.b0 + (turn - na)) * kTile;
      const typename Op::KvTile kt(kr, key0, a.Lk, HS * (int)sizeof(T)), vt(vr, key0, a.Lk, HS * (int)sizeof(T));
      if (kt.whole) op.template load_tile<true>(kt, vt, lane);   // (K and V are cut into shards alike)
      else op.template load_tile<false>(kt, vt, lane);
      op.stash_k(lds, lane);
      if constexpr (sizeof(T) == 4 && HS == 128) {
        if (kt.whole) op.template load_v<true>(vt, lane);
        else op.template load_v<false>(vt, lane);
      }   // K, V, Q and O together are more than the registers
      f32x16 s = op.scores(lds, lane);
      const bool need_mask = key0 + kTile > a.Lk || (a.causal && pos_max(kpos, key0, min(a.Lk, key0 + kTile)) > qmin);
      if (need_mask) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = key0 + 8 * (e >> 2) + 4 * hl + (e & 3);
          const bool vis = key < a.Lk && (!a.causal || pos_of(kpos, key) <= qp);
          s[e] = vis ? s[e] : -INFINITY;
        }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[e]);
      mx = both_halves_max(mx);
      if (!shared_first) {
        int t = lane;   // places in LDS derived here, from a lane index the compiler cannot see through: kept, they are spilled
        asm volatile("" : "+v"(t));
        if (wave < 2 && t < 32) first_s[wave][t] = (wave == 0 || i == 0) ? mx : -INFINITY;
        __syncthreads();
        m = fmaxf(first_s[0][t & 31], first_s[1][t & 31]);
        if constexpr (STATE) {   // (a row that has a state goes on from its maximum)
          const float ms = m_state_s[t & 31];
          m = ms > -INFINITY ? ms : m;
        }
        shared_first = true;
      }
      if (__any((mx - m) * a.scale_log2 > kRescaleThreshold)) {   // (m = -inf and a key: inf; no key at all: NaN, no)
        const float m_new = fmaxf(m, mx);
        const float alpha = __builtin_amdgcn_exp2f(m * a.scale_log2 - (m_new == -INFINITY ? 0.f : m_new * a.scale_log2));   // m = -inf -> 0
        l *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
        m = m_new;
      }
      const float mc = m == -INFINITY ? 0.f : m * a.scale_log2;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        s[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], a.scale_log2, -mc));
        l += s[e];
      }
      op.accumulate(s, o, lds, lane);
    }
    turn -= nt;
  }
  if (!shared_first) {   // no tile for this wave
    if (wave < 2 && lane < 32) first_s[wave][lane] = -INFINITY;
    __syncthreads();
  }

  // ---- the waves' states are combined: common maximum, scaled outputs side by side in LDS, summed row by row
  int end_lane = lane;   // (a lane index of its own for the epilogue: what derives from it is not kept across the loop)
  asm volatile("" : "+v"(end_lane));
  constexpr int PER_ROW = HS / 4, ROWS_PER_PASS = kWaves * 64 / PER_ROW, PASSES = kRows / ROWS_PER_PASS;
  // where the record holds dims 4 c .. 4 c + 3 of row rr: this thread's part of the last step
  auto rec_at = [&](int rr, int c) { return rec + ((c >> 1) * 64 + (c & 1) * 32 + rr) * 4; };
  f32x4 o_state[STATE ? PASSES : 1];
  if constexpr (STATE) {   // asked for here, needed behind two barriers
    if (!a.state_first) {
#pragma unroll
      for (int pass = 0; pass < PASSES; ++pass)
        o_state[pass] = *(const f32x4*)rec_at(pass * ROWS_PER_PASS + (int)threadIdx.x / PER_ROW, (int)threadIdx.x % PER_ROW);
    }
  }
  l = both_halves_sum(l);
  if (end_lane < 32) {
    m_s[wave][(end_lane & 31)] = m;
    l_s[wave][(end_lane & 31)] = l;
  }
  __syncthreads();
  // (every loop over the waves is unrolled, all its LDS reads in flight at once: a wave that had no tile adds zeros)
  float mw[kWaves], m_all = -INFINITY;
#pragma unroll
  for (int j = 0; j < kWaves; ++j) mw[j] = m_s[j][(end_lane & 31)];
#pragma unroll
  for (int j = 0; j < kWaves; ++j) m_all = fmaxf(m_all, mw[j]);
  if constexpr (STATE) m_all = fmaxf(m_all, m_state_s[end_lane & 31]);
  const float mc = m_all == -INFINITY ? 0.f : m_all * a.scale_log2;
  {
    const float f = __builtin_amdgcn_exp2f(m * a.scale_log2 - mc);
    float* dst = (float*)smem + (wave * kRows + (end_lane & 31)) * OSTR;
#pragma unroll
    for (int gi = 0; gi < Op::kGroups; ++gi) *(f32x4*)(dst + Op::group_dim(gi, end_lane >> 5)) = Op::group(o, gi) * f;
  }
  if (wave == 0 && (STATE || end_lane < 32)) {
    float tot = 0.f;
#pragma unroll
    for (int j = 0; j < kWaves; ++j) tot += l_s[j][(end_lane & 31)] * __builtin_amdgcn_exp2f(mw[j] * a.scale_log2 - mc);
    if constexpr (STATE) {
      float f = 0.f;
      float* const lane_rec = rec + HS * kRows;   // m of 64 lanes, l of 64 lanes: a row's l is the sum of its two
      if (!a.state_first) {
        f = __builtin_amdgcn_exp2f(m_state_s[end_lane & 31] * a.scale_log2 - mc);
        tot += (lane_rec[64 + (end_lane & 31)] + lane_rec[96 + (end_lane & 31)]) * f;
      }
      f_state_s[end_lane & 31] = f;
      if (!a.state_last) {
        lane_rec[end_lane] = m_all;
        lane_rec[64 + end_lane] = end_lane < 32 ? tot : 0.f;
      }
    }
    if (!STATE || a.state_last) {
      inv_s[(end_lane & 31)] = tot > 0.f ? 1.f / tot : 0.f;   // a row that saw no key: O = 0, LSE = -inf
      if (row0 + (end_lane & 31) < a.Lq)
        a.lse[(((int64_t)rank * a.bs + b) * a.hq + h) * a.Lq + row0 + (end_lane & 31)] = tot > 0.f ? m_all * a.scale + logf(tot) : -INFINITY;
    }
  }
  __syncthreads();
  const BlockRows orow = block_rows(a.o, sizeof(OutT), HS, a.bs, a.n_q, a.q_heads, r * a.U, b, u * a.hq + h);
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    const int rr = pass * ROWS_PER_PASS + (int)threadIdx.x / PER_ROW, c = (int)threadIdx.x % PER_ROW;
    const float* src = (const float*)smem + rr * OSTR + 4 * c;
    f32x4 sum = *(const f32x4*)src;
#pragma unroll
    for (int j = 1; j < kWaves; ++j) sum += *(const f32x4*)(src + j * (kRows * OSTR));
    if constexpr (STATE) {
      if (!a.state_first) sum += o_state[pass] * f_state_s[rr];
      if (!a.state_last) {
        *(f32x4*)rec_at(rr, c) = sum;
        continue;
      }
    }
    sum *= inv_s[rr];
    if (row0 + rr < a.Lq) {
      OutT* dst = (OutT*)orow.row(row0 + rr) + 4 * c;
      if constexpr (sizeof(OutT) == 4) *(f32x4_any*)dst = sum;
      else *(u32x2_any*)dst = u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
    }
  }
}

template <typename T, int HS, typename OutT, bool STATE = false>
int launch_typed(WsArgs a, int64_t grid, hipStream_t stream) {
  constexpr size_t lds = lds_bytes<T, HS>();
  auto kern = wave_split_attn_fwd<T, HS, OutT, STATE>;
  static LdsLimitRaised lds_limit;   // per kernel instance
  if (!raise_dynamic_lds_limit((const void*)kern, lds, lds_limit)) return USP_ERR_LAUNCH;
  const int64_t at_once = max_workgroups(kWaves * 64);
  for (int64_t first = 0; first < grid; first += at_once) {
    a.first_wg = (int)first;
    hipLaunchKernelGGL(kern, dim3((unsigned)std::min(grid - first, at_once)), dim3(kWaves * 64), lds, stream, a);
    const int st = launch_status();
    if (st != USP_OK) return st;
  }
  return USP_OK;
}

int launch(WsArgs a, int hs, int in_dtype, int o_dtype, hipStream_t stream) {
  a.g = a.hq / a.hkv;
  a.by_hkv = fast_div(a.hkv); a.by_bs = fast_div(a.bs); a.by_ranks = fast_div(a.n_ranks);
  a.by_g = fast_div(a.g); a.by_U = fast_div(a.U);
  a.n_qtiles = (a.Lq + kRows - 1) / kRows;
  a.scale_log2 = a.scale * 1.4426950408889634f;
  const int64_t grid = (int64_t)a.n_qtiles * a.hq * a.bs * a.n_ranks;
  if (grid > 0x7fffffffll) return USP_ERR_UNSUPPORTED;
  if (a.state) {   // bf16 data
    if (hs == 128) return o_dtype == USP_FP32 ? launch_typed<__bf16, 128, float, true>(a, grid, stream) : launch_typed<__bf16, 128, __bf16, true>(a, grid, stream);
    return o_dtype == USP_FP32 ? launch_typed<__bf16, 64, float, true>(a, grid, stream) : launch_typed<__bf16, 64, __bf16, true>(a, grid, stream);
  }
  if (in_dtype == USP_FP32) {
    if (hs == 128) return o_dtype == USP_FP32 ? launch_typed<float, 128, float>(a, grid, stream) : launch_typed<float, 128, __bf16>(a, grid, stream);
    return o_dtype == USP_FP32 ? launch_typed<float, 64, float>(a, grid, stream) : launch_typed<float, 64, __bf16>(a, grid, stream);
  }
  if (hs == 128) return o_dtype == USP_FP32 ? launch_typed<__bf16, 128, float>(a, grid, stream) : launch_typed<__bf16, 128, __bf16>(a, grid, stream);
  return o_dtype == USP_FP32 ? launch_typed<__bf16, 64, float>(a, grid, stream) : launch_typed<__bf16, 64, __bf16>(a, grid, stream);
}

}  // namespace

int launch_wave_split_usp_fwd(const usp_problem& p, const void* q, const void* k, const void* v, void* o, float* lse,
                              int rank_begin, int rank_end, float scale, hipStream_t stream) {
  WsArgs a = {};
  a.q = q; a.k = k; a.v = v; a.o = o; a.lse = lse;
  a.bs = p.bs; a.hq = p.hc / p.ulysses; a.hkv = p.hk / p.ulysses;
  a.q_heads = p.hc; a.kv_heads = p.hk;
  a.U = p.ulysses; a.R = p.ring; a.rank_begin = rank_begin; a.n_ranks = rank_end - rank_begin;
  a.n_q = a.n_k = fast_div(p.L / ((int64_t)p.ulysses * p.ring));
  a.Lq = a.Lk = (int)(p.L / p.ring);
  a.causal = p.causal ? 1 : 0; a.split = p.split;
  a.scale = scale;
  return launch(a, p.hs, p.dtype, p.dtype, stream);
}

int launch_wave_split_block_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int bs, int64_t Lq,
                                int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc& qpos,
                                const usp_posdesc& kpos, int in_dtype, int o_dtype, hipStream_t stream, const RingState* state) {
  WsArgs a = {};
  a.q = q; a.k = k; a.v = v; a.o = o; a.lse = lse;
  a.bs = bs; a.hq = a.q_heads = hq; a.hkv = a.kv_heads = hkv;
  a.U = a.R = a.n_ranks = 1;
  a.Lq = (int)Lq; a.n_q = fast_div(Lq);
  a.Lk = (int)Lk; a.n_k = fast_div(Lk);
  a.causal = causal; a.split = -1;
  if (state) {
    a.state = state->state; a.state_first = state->first; a.state_last = state->last;
    a.state_records = (int)((Lq + 255) / 256) * 8;
  }
  a.qpos = PosDesc32{(int)qpos.start0, (int)qpos.len0, (int)qpos.start1, (int)qpos.len1};
  a.kpos = PosDesc32{(int)kpos.start0, (int)kpos.len0, (int)kpos.start1, (int)kpos.len1};
  a.scale = scale;
  return launch(a, hs, in_dtype, o_dtype, stream);
}

}  // namespace usp
