// Attention forward with the keys of 32 query rows split over the eight waves of ONE workgroup: the whole ring loop of
// Algorithm 1 (all-to-alls, blocks, merge) for a range of virtual ranks in a single launch, for the problems where
// launches and latency are the time rather than the matrix core, and for fp32 data of every size.
//
//   * A workgroup owns 32 query rows (16 in small fp32 grids) of one (rank, batch, head).  Its waves take the visible 32-key tiles of all K/V
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
// What bounds it.  Small problems: the chain of one workgroup.  Time stamps in a workgroup of one tile per wave (fp32, head
// size 64, 19 thousand cycles): 5 to 7 thousand before the first product, most of it loads waiting to issue: what a CU loads
// goes through one path of 64 bytes a cycle, and the eight waves each loaded all of Q (a third of everything) and had their
// V in front of the others' K.  So Q is loaded once and shared through LDS, V is asked for behind the barrier that this
// needs anyway, and the next tile's K and V while a tile is worked on (a tile of a walk took 3.3 thousand cycles with its
// loads waited for).  All that does not depend on the workgroup is worked out on the host.  Together: four fp32 ranks of
// L = 256 9.3 -> 8.6 us (6.5 with 16 rows per workgroup, wave_split_fp32_rows()), four bf16 ranks of L = 1024 12.1 -> 10.9, one of
// eight ranks of L = 2048 (32 heads on 8) 18.7 -> 16.6, all eight 90.6 -> 79.0, fp32 at L = 2048 (eight heads of size 64, two ranks a ring) 47.1 -> 43.0.
// Large problems: every workgroup reads all its keys for only 32 rows, eight times the L2 and LDS traffic per product of the
// 256-row kernel.  Where the line between the two lies is in usp_api.cpp (short_in_one_launch).  fp32: the matrix core at
// fp32 rate, 125 TFLOP/s at L = 2048, four heads of size 128, no mask (154 is what a large fp32 matrix product reaches).
#include <algorithm>

#include "attn_device.h"
#include "usp_internal.h"

namespace usp {
namespace {

using namespace dev;

constexpr int kWaves = kWaveSplitWaves, kTile = kWaveSplitTile;

// Where the positions of ring block r begin: those of its two runs are start0 + r step0 .. and start1 - r step1 ..
// (Algorithm 2: chunks r and 2R-1-r of 2R, or block r of R; one given block: steps of 0; no mask: one run from 0).
struct BlockPositions {
  int start0, step0, len0, start1, step1, len1;
  __device__ PosDesc32 of(int r) const { return PosDesc32{start0 + r * step0, len0, start1 - r * step1, len1}; }
};

// The keys of a ring block (one batch entry) lie in the shards [U][bs][n][heads][hs], row j at j rows and (j / n) jumps from
// the block's first.  Every tile is read through buffer descriptors (K, V) whose extent ends with its last row: rows past it
// read as zeros.  The row within the tile is part of the vector offset, which the descriptor's range check covers (the scalar
// offset it does not).  With a second path for tiles that cross from one shard into the next, and a branch round the loads
// where there is no next tile, every wait for one tile's loads was a wait for all that were in flight.  So either tiles are
// numbered shard by shard and none crosses, or, in instances of their own, all may: see wave_split_crossing().  With a batch
// of one a block is one run of n = Lk rows.
struct KeyTiles {
  FastDiv by_n, by_tiles;      // rows of a shard; tiles of a shard
  int one;                     // tiles are numbered through: a single run of rows, or tiles that cross
  __device__ int upto(int keys) const {   // tiles that hold the first `keys` keys
    if (one) return (unsigned)(keys + kTile - 1) / kTile;
    const int shard = by_n.split(keys);
    return shard * (int)by_tiles.d + (int)((unsigned)(keys + kTile - 1) / kTile);
  }
  __device__ int of(int key) const {
    if (one) return (unsigned)key / kTile;
    const int shard = by_n.split(key);
    return shard * (int)by_tiles.d + (int)((unsigned)key / kTile);
  }
};

// Everything that does not depend on the workgroup is worked out on the host: of the 19 thousand cycles that a workgroup of
// one tile per wave took, 6 thousand went by before its first product, in 500 instructions of addresses and positions.
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
  FastDiv n_q;                // rows of a Q shard
  KeyTiles tiles;
  FastDiv by_hkv, by_bs, by_ranks, by_g, by_U;
  int Lq, Lk;                 // rows of a ring block
  int n_qtiles, causal;
  // elements from one ring block to the next, from one batch entry to the next, and what rows of the next shard lie further
  // on than the next row would (0: a batch of one)
  uint64_t q_ring, q_run, q_jump, kv_ring, kv_run, kv_jump;
  BlockPositions qpos, kpos;
  float scale, scale_log2;
  // Running state of a ring that delivers its blocks one per call (STATE instances), in the 256-row kernel's records
  // (block_attn_fwd.hip): per 32 rows of a (batch, head) the O^T accumulator as [hs / 8][64 lanes][4], m, and l, per lane.
  float* state;
  int state_first, state_last, state_records;   // records of a (batch, head)
};

__device__ inline uint64_t times(int n, uint64_t x) { return (uint64_t)(uint32_t)n * x; }

// What a tile that crosses knows besides: rows from `cross` on lie `jump` bytes further on; or, for any number of crossings, the
// bytes from the tile's first row to row lane % 32, handed from lane to lane where the rows are loaded.
template <int CROSS> struct Crossing {};
template <> struct Crossing<kOneCross> { int cross, jump; };
template <> struct Crossing<kAnyCross> { int row_at; };
template <int CROSS> struct Tile : Crossing<CROSS> {
  uint64_t at;          // bytes from the tensor's begin to the tile's first row
  int row_bytes, extent;
  int key0, end;        // its keys
  // (!exists: no tile; its loads find nothing in range and give zeros)
  __device__ Tile(const KeyTiles& tiles, bool exists, int t, int Lk, uint64_t block, uint64_t jump_, int row_bytes_, int row_len) : row_bytes(row_bytes_) {
    key0 = t * kTile;
    end = min(key0 + kTile, Lk);
    at = block;
    if constexpr (CROSS != kNoCross) {
      int in_shard = key0;
      at += times(tiles.by_n.split(in_shard), jump_) + (uint64_t)(uint32_t)key0 * (uint32_t)row_bytes;
      const int last = end - 1 - key0, jump = (int)jump_;
      extent = last * row_bytes + row_len;
      if constexpr (CROSS == kOneCross) {
        this->cross = (int)tiles.by_n.d - in_shard;
        this->jump = jump;
        extent += last >= this->cross ? jump : 0;
      } else {
        extent += tiles.by_n.div(in_shard + last) * jump;
        // (the thread's number, not a lane index from the caller: that, passed through, made every instance longer by 10 to 30
        // instructions; four bf16 ranks of L = 1024 10.93 us for 10.87)
        const int row = (int)threadIdx.x % kTile;
        this->row_at = row * row_bytes + tiles.by_n.div(in_shard + row) * jump;
      }
      extent = exists ? extent : 0;
      return;
    }
    if (!tiles.one) {
      const int shard = tiles.by_tiles.split(t);
      key0 = shard * (int)tiles.by_n.d + t * kTile;
      end = min(key0 + kTile, (shard + 1) * (int)tiles.by_n.d);
      at += times(shard, jump_);
    }
    at += (uint64_t)(uint32_t)key0 * (uint32_t)row_bytes;
    extent = exists ? (end - 1 - key0) * row_bytes + row_len : 0;
  }
  // x[i] = 16 bytes (8: V of the fp32 kernel at head size 64) at byte `col` of row lane_row + step(i).  kApart: tiles that do
  // not cross have their loads to themselves, for instances that wait for all of a tile's loads anyway.
  template <bool kApart = false, typename V, int N, typename Step>
  __device__ void load(V (&x)[N], const void* tensor, int lane_row, Step step, int col) const {
    if constexpr (kApart && CROSS == kOneCross) {
      if (this->cross >= kTile) {
        load_from<kNoCross>(x, tensor, lane_row, step, col);
        return;
      }
    }
    load_from<CROSS>(x, tensor, lane_row, step, col);
  }
  template <int HOW, typename V, int N, typename Step>
  __device__ void load_from(V (&x)[N], const void* tensor, int lane_row, Step step, int col) const {
    static_assert(sizeof(V) == 16 || sizeof(V) == 8, "");
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((char*)tensor + at, 0, extent, kRawBufferFlags);
    const int voff0 = lane_row * row_bytes + col;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int voff = voff0 + step(i) * row_bytes;
      if constexpr (HOW == kOneCross) voff += lane_row >= this->cross - step(i) ? this->jump : 0;
      if constexpr (HOW == kAnyCross) voff = __builtin_amdgcn_ds_bpermute((lane_row + step(i)) * 4, this->row_at) + col;
      if constexpr (sizeof(V) == 16) x[i] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, 0, 0));
      else x[i] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(rsrc, voff, 0, 0));
    }
  }
};

// ---- operands of one data type: the fragments of Q and of a 32-key tile, and the two products -------------------
// What a 32-row workgroup's lanes hold: lane = row l32 (column of S^T and O^T); score e is key first_key() + key_step(e).
struct Rows32 {
  static constexpr int kRows = 32, kScores = 16;
  typedef f32x16 Scores;
  typedef f32x16 Acc;
  static __device__ int row_of(int lane) { return lane & 31; }
  static __device__ int first_key(int lane) { return 4 * (lane >> 5); }
  static constexpr __device__ int key_step(int e) { return 8 * (e >> 2) + (e & 3); }
  static __device__ float max_of_row(float x) { return both_halves_max(x); }
  static __device__ float sum_of_row(float x) { return both_halves_sum(x); }
};
// ... and a 16-row one's (fp32): four lanes to a row, 16 lanes apart.
struct Rows16 {
  static constexpr int kRows = 16, kScores = 8;
  typedef float Scores __attribute__((ext_vector_type(8)));
  typedef f32x4 Acc;
  static __device__ int row_of(int lane) { return lane & 15; }
  static __device__ int first_key(int lane) { return 4 * (lane >> 4); }
  static constexpr __device__ int key_step(int e) { return 16 * (e >> 2) + (e & 3); }
  static __device__ u32x2 other(float x) {   // x of this quarter and of the one 16 lanes off
    const uint32_t xi = __builtin_bit_cast(uint32_t, x);
    return __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
  }
  static __device__ float max_of_row(float x) {
    const u32x2 r = other(x);
    const uint32_t a = r[0], b = r[1];
    return both_halves_max(fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)));
  }
  static __device__ float sum_of_row(float x) {
    const u32x2 r = other(x);
    const uint32_t a = r[0], b = r[1];
    return both_halves_sum(__builtin_bit_cast(float, a) + __builtin_bit_cast(float, b));
  }
};

template <typename T, int HS, int ROWS, int CROSS> struct Operands;

template <int HS, int CROSS> struct Operands<__bf16, HS, 32, CROSS> : Rows32 {
  static constexpr int kBlocks = HS / 32;   // accumulators
  static constexpr int KSTEPS = HS / 16, DB = HS / 32, CPR = HS / 8;
  static constexpr int kWavesPerSimd = HS == 64 ? 4 : 2;   // head size 64: two workgroups to a CU
  // Q fragments: kept in registers, or, where four waves to a SIMD leave none to spare, read from LDS for every tile.
  static constexpr bool kQInRegs = HS == 128;
  static constexpr bool kAhead = true;     // a tile's K and V are asked for while the tile before is worked on
  // Rows of the wave's LDS tile.  K: an odd number of 16-byte chunks, no bank conflicts on the fragment reads; V: an odd
  // multiple of 64 bytes, none on the transpose reads.  K and V take turns in one tile (a wave's LDS accesses are in order).
  static constexpr int KSTR = HS * 2 + 48, VSTR = HS * 2 + 64, QSTR = HS * 2 + 16;
  static constexpr int kLdsPerWave = kTile * VSTR;
  static constexpr int TL = kTile * CPR / 64;            // 16-byte loads per lane of a tile
  bf16x8 q[kQInRegs ? KSTEPS : 1];
  u32x4 k[TL], v[TL];

  __device__ static bf16x8 q_at(const char* q_lds, int lane, int ks) {
    return *(const bf16x8*)(q_lds + (lane & 31) * QSTR + 32 * ks + 16 * (lane >> 5));
  }
  __device__ void read_q(const char* q_lds, int lane) {
    if constexpr (kQInRegs) {
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) q[ks] = q_at(q_lds, lane, ks);
    }
  }
  template <typename Tile> __device__ static void load_rows(u32x4 (&t)[TL], const void* tensor, const Tile& tile, int lane) {
    tile.load(t, tensor, lane / CPR, [](int c) { return c * (64 / CPR); }, (lane % CPR) * 16);
  }
  template <int STR> __device__ static void stash_rows(char* lds, const u32x4 (&t)[TL], int lane) {
#pragma unroll
    for (int c = 0; c < TL; ++c) {
      const int ch = lane + 64 * c;
      *(u32x4*)(lds + (ch / CPR) * STR + (ch % CPR) * 16) = t[c];
    }
    __builtin_amdgcn_wave_barrier();   // this wave's own LDS accesses stay in this order
  }
  template <typename Tile> __device__ void load_k(const void* tensor, const Tile& t, int lane) { load_rows(k, tensor, t, lane); }
  template <typename Tile> __device__ void load_v(const void* tensor, const Tile& t, int lane) { load_rows(v, tensor, t, lane); }
  __device__ void stash_k(char* lds, int lane) { stash_rows<KSTR>(lds, k, lane); }
  // S^T = K Q^T; leaves V in the LDS tile
  __device__ f32x16 scores(char* lds, const char* q_lds, int lane) {
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    const char* row = lds + (lane & 31) * KSTR + 16 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(row + 32 * ks), kQInRegs ? q[kQInRegs ? ks : 0] : q_at(q_lds, lane, ks), s, 0, 0, 0);
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
  static __device__ int group_dim(int gi, int lane) { return dim4(gi / 4, gi % 4, lane >> 5); }
  static __device__ f32x4 group(const f32x16 (&o)[DB], int gi) { return out4(o, gi / 4, gi % 4); }
};

template <int HS, int CROSS> struct Operands<float, HS, 32, CROSS> : Rows32 {
  static constexpr int kBlocks = HS / 32;
  static constexpr int DB = HS / 32, KC = HS / 8, CPR = HS / 4;
  static constexpr int kWavesPerSimd = 2;
  // (Head size 128: Q, K, V and O are all the registers.  With Q read from LDS for every tile there is room for the next K, and
  // it was slower: 72.4 us for 68.7 at L = 2048, four heads, no mask.)
  static constexpr bool kAhead = HS == 64;
  static constexpr int KSTR = HS * 4 + 16, QSTR = KSTR;  // an odd number of 16-byte chunks
  static constexpr int kLdsPerWave = kTile * KSTR;
  static constexpr int TL = kTile * CPR / 64;
  // (... and where the rows' offsets want registers, most of Q is read from LDS for every tile.)
  static constexpr int kQInRegs = HS == 128 && CROSS == kAnyCross ? KC - 10 : KC;
  typedef float vrow __attribute__((ext_vector_type(DB)));
  f32x4 q[kQInRegs];     // dims 8 c + 4 (lane half) .. + 3: the product's two k indices are the lane halves
  f32x4 k[TL];           // a tile's K rows on their way to LDS
  vrow v[16];            // V of the key that score register i of this lane half holds, dims DB l32 .. + DB - 1

  __device__ static f32x4 q_at(const char* q_lds, int lane, int c) {
    return *(const f32x4*)(q_lds + (lane & 31) * QSTR + 32 * c + 16 * (lane >> 5));
  }
  __device__ void read_q(const char* q_lds, int lane) {
#pragma unroll
    for (int c = 0; c < kQInRegs; ++c) q[c] = q_at(q_lds, lane, c);
  }
  template <typename Tile> __device__ void load_k(const void* tensor, const Tile& t, int lane) {
    t.template load<!kAhead>(k, tensor, lane / CPR, [](int c) { return c * (64 / CPR); }, (lane % CPR) * 16);
  }
  template <typename Tile> __device__ void load_v(const void* tensor, const Tile& t, int lane) {
    t.template load<!kAhead>(v, tensor, 4 * (lane >> 5), [](int i) { return 8 * (i >> 2) + (i & 3); }, (lane & 31) * (DB * 4));
  }
  __device__ void stash_k(char* lds, int lane) {
#pragma unroll
    for (int c = 0; c < TL; ++c) {
      const int ch = lane + 64 * c;
      *(f32x4*)(lds + (ch / CPR) * KSTR + (ch % CPR) * 16) = k[c];
    }
    __builtin_amdgcn_wave_barrier();
  }
  __device__ f32x16 scores(char* lds, const char* q_lds, int lane) {
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    const char* row = lds + (lane & 31) * KSTR + 16 * (lane >> 5);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const f32x4 kc = *(const f32x4*)(row + 32 * c), qc = c < kQInRegs ? q[c < kQInRegs ? c : 0] : q_at(q_lds, lane, c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float ka = kc[e], qa = qc[e];
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
  static __device__ int group_dim(int gi, int lane) {
    const int hl = lane >> 5, r = DB == 4 ? gi : 2 * gi;                 // the product rows of this group: one (DB = 4) or two (DB = 2)
    return DB * (8 * (r >> 2) + 4 * hl + (r & 3));
  }
  static __device__ f32x4 group(const f32x16 (&o)[DB], int gi) {
    if constexpr (DB == 4) return f32x4{o[0][gi], o[1][gi], o[2][gi], o[3][gi]};
    else return f32x4{o[0][2 * gi], o[1][2 * gi], o[0][2 * gi + 1], o[1][2 * gi + 1]};
  }
};

// fp32, 16 rows per workgroup, v_mfma_f32_16x16x4_f32: for grids that leave half the chip idle, and where the matrix core at
// fp32 rate is the longest part of a workgroup's time (rule in wave_split_fp32_rows()).  Four k indices: the lane quarters.
template <int HS, int CROSS> struct Operands<float, HS, 16, CROSS> : Rows16 {
  static constexpr int NB = HS / 16, VH = NB / 4, KC = HS / 16, CPR = HS / 4;
  static constexpr int kBlocks = NB;
  static constexpr int kWavesPerSimd = 2;
  static constexpr bool kAhead = true;
  static constexpr int KSTR = HS * 4 + 16, QSTR = KSTR;
  static constexpr int kLdsPerWave = kTile * KSTR;
  static constexpr int TL = kTile * CPR / 64;
  f32x4 q[KC];           // dims 16 c + 4 (lane quarter) .. + 3
  f32x4 k[TL];
  f32x4 v[VH][8];        // V of the key of score e, dims NB (lane & 15) + 4 half .. + 3

  __device__ void read_q(const char* q_lds, int lane) {
#pragma unroll
    for (int c = 0; c < KC; ++c) q[c] = *(const f32x4*)(q_lds + (lane & 15) * QSTR + 64 * c + 16 * (lane >> 4));
  }
  template <typename Tile> __device__ void load_k(const void* tensor, const Tile& t, int lane) {
    t.load(k, tensor, lane / CPR, [](int c) { return c * (64 / CPR); }, (lane % CPR) * 16);
  }
  template <typename Tile> __device__ void load_v(const void* tensor, const Tile& t, int lane) {
#pragma unroll
    for (int half = 0; half < VH; ++half)
      t.load(v[half], tensor, first_key(lane), [](int e) { return key_step(e); }, (lane & 15) * (NB * 4) + 16 * half);
  }
  __device__ void stash_k(char* lds, int lane) {
#pragma unroll
    for (int c = 0; c < TL; ++c) {
      const int ch = lane + 64 * c;
      *(f32x4*)(lds + (ch / CPR) * KSTR + (ch % CPR) * 16) = k[c];
    }
    __builtin_amdgcn_wave_barrier();
  }
  __device__ Scores scores(char* lds, const char*, int lane) {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;   // keys 0 .. 15 and 16 .. 31
    const char* row = lds + (lane & 15) * KSTR + 16 * (lane >> 4);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const f32x4 k0 = *(const f32x4*)(row + 64 * c), k1 = *(const f32x4*)(row + 16 * KSTR + 64 * c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a0 = k0[e], a1 = k1[e], qa = q[c][e];
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, qa, s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, qa, s1, 0, 0, 0);
      }
    }
    __builtin_amdgcn_wave_barrier();
    return __builtin_shufflevector(s0, s1, 0, 1, 2, 3, 4, 5, 6, 7);
  }
  __device__ void accumulate(const Scores& p, Acc (&o)[NB], const char*, int) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float pe = p[e];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const float va = v[nb / 4][e][nb % 4];
        o[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(va, pe, o[nb], 0, 0, 0);
      }
    }
  }
  // register i of block nb is head dim NB (4 (lane quarter) + i) + nb
  static constexpr int kGroups = NB;
  static __device__ int group_dim(int gi, int lane) { return NB * (4 * (lane >> 4) + gi / VH) + 4 * (gi % VH); }
  static __device__ f32x4 group(const Acc (&o)[NB], int gi) {
    const int i = gi / VH, b = 4 * (gi % VH);
    return f32x4{o[b][i], o[b + 1][i], o[b + 2][i], o[b + 3][i]};
  }
};

template <typename T, int HS, int ROWS>
constexpr size_t lds_bytes() {
  const size_t states = (size_t)kWaves * ROWS * (HS + 4) * sizeof(float);
  const size_t tiles = (size_t)kWaves * Operands<T, HS, ROWS, kNoCross>::kLdsPerWave + ROWS * Operands<T, HS, ROWS, kNoCross>::QSTR;
  return (states > tiles ? states : tiles);
}

template <typename T, int HS, typename OutT, bool STATE = false, int ROWS = 32, int CROSS = kNoCross>
__global__ __attribute__((amdgpu_flat_work_group_size(kWaves * 64, kWaves * 64), amdgpu_waves_per_eu(Operands<T, HS, ROWS, CROSS>::kWavesPerSimd, Operands<T, HS, ROWS, CROSS>::kWavesPerSimd)))
void wave_split_attn_fwd(const WsArgs a) {
  using Op = Operands<T, HS, ROWS, CROSS>;
  static_assert(!STATE || ROWS == 32, "the state's records are of 32 rows");
  constexpr int NB = Op::kBlocks, kRows = ROWS, OSTR = HS + 4;   // floats between the rows of a state in LDS: an odd number of 16 B chunks
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ float m_s[kWaves][kRows], l_s[kWaves][kRows], inv_s[kRows], first_s[2][kRows];
  const int lane = threadIdx.x & 63;
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
  constexpr int kNever = 0x7ffffffe;   // no mask: a query after every key
  const PosDesc32 qpos = a.qpos.of(r);
  const int qmin = a.causal ? pos_min(qpos, row0, row1) : kNever, qmax = a.causal ? pos_max(qpos, row0, row1) : kNever;

  Op op;
  // (element offsets: Q and O lie alike, whatever their types; K and V too)
  const uint64_t q_at = times(r, a.q_ring) + times(b, a.q_run) + (uint32_t)((u * a.hq + h) * HS);
  const uint64_t kv_at = times(b, a.kv_run) + (uint32_t)((u * a.hkv + kvh) * HS);
  auto q_row = [&](int j) { return q_at + (uint64_t)(uint32_t)j * (uint32_t)(a.q_heads * HS) + (a.q_jump ? times(a.n_q.div(j), a.q_jump) : 0); };
  // Q is read once and shared through LDS: loaded by every wave for itself, it was a third of what a workgroup with one tile
  // per wave moves through the CU's load path (64 bytes a cycle), ahead of all of its K.
  constexpr int QCH = HS * (int)sizeof(T) / 16, QL = kRows * QCH / (kWaves * 64);   // 16-byte chunks of a row; of a thread
  char* const q_lds = smem + kWaves * Op::kLdsPerWave;
  u32x4 qreg[QL > 0 ? QL : 1];
  const bool q_loader = QL > 0 || (int)threadIdx.x < kRows * QCH;
  if (q_loader) {
#pragma unroll
    for (int i = 0; i < (QL > 0 ? QL : 1); ++i) {
      const int ch = (int)threadIdx.x + i * (kWaves * 64), row = min(row0 + ch / QCH, a.Lq - 1);
      qreg[i] = *(const u32x4_any*)((const char*)a.q + q_row(row) * sizeof(T) + (ch % QCH) * 16);
    }
  }

  typename Op::Acc o[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < (int)(sizeof(o[0]) / 4); ++i) o[nb][i] = 0.f;
  float m = -INFINITY, l = 0.f;

  // The walk over the blocks' visible tiles, this wave's every eighth.  (Algorithm 1 step 5: step i visits block (r - i) mod R.)
  // Of every ascending run of key positions the visible ones are a prefix: of tiles 0 .. and of tiles from the second run's on.
  int step = -1, kstart0 = 0, kstart1 = 0, na = 0, skip = 0, nt = 0;
  uint64_t block_at = 0;
  auto visible = [&](int blk) {
    const PosDesc32 kp = a.kpos.of(blk);
    kstart0 = kp.start0;
    kstart1 = kp.start1;
    const int c0 = min(max(qmax - kp.start0, -1), kp.len0 - 1) + 1, c1 = min(max(qmax - kp.start1, -1), kp.len1 - 1) + 1;
    na = a.tiles.upto(c0);
    const int b0 = max(a.tiles.of(kp.len0), na);
    skip = b0 - na;
    nt = na + (c1 > 0 ? max(a.tiles.upto(kp.len0 + c1) - b0, 0) : 0);
  };

  // The state enters with the merge, as a ninth wave's would, and leaves from there: nothing of it is held meanwhile.
  float* rec = nullptr;
  __shared__ float m_state_s[kRows], f_state_s[kRows];
  if constexpr (STATE) {
    rec = a.state + ((size_t)(b * a.hq + h) * a.state_records + row0 / kRows) * (HS * kRows + 128);
    if (!a.state_first && !a.state_last) {   // rows that see nothing of this block: their state stays as it is
      visible(0);
      if (nt == 0) return;   // workgroup-uniform
      nt = 0;                // (the walk has not begun)
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
  auto next_tile = [&]() {   // of the walk; false: it has ended
    while (turn >= nt) {
      turn -= nt;
      if (++step >= a.R) return false;
      const int blk = r - step + (r < step ? a.R : 0);
      visible(blk);
      block_at = kv_at + times(blk, a.kv_ring);
    }
    return true;
  };
  const int row_bytes = a.kv_heads * HS * (int)sizeof(T);
  auto tile_now = [&](bool exists) {
    return Tile<CROSS>(a.tiles, exists, turn < na ? turn : turn + skip, a.Lk, block_at * sizeof(T), a.kv_jump * sizeof(T), row_bytes, HS * (int)sizeof(T));
  };
  bool more = next_tile();
  // Loads of a tile to come are always issued, with or without one: with a branch round them, what waits for older loads would
  // have to wait for all.
  Tile<CROSS> tile = tile_now(more);
  if (Op::kAhead) op.load_k(a.k, tile, lane);
  if (q_loader) {
#pragma unroll
    for (int i = 0; i < (QL > 0 ? QL : 1); ++i) {
      const int ch = (int)threadIdx.x + i * (kWaves * 64);
      *(u32x4*)(q_lds + (ch / QCH) * Op::QSTR + (ch % QCH) * 16) = qreg[i];
    }
  }
  __syncthreads();
  if (Op::kAhead) op.load_v(a.v, tile, lane);   // (behind every wave's K)
  op.read_q(q_lds, lane);
  while (more) {
    const int key0 = tile.key0, key_end = tile.end, start0 = kstart0, start1 = kstart1;
    const bool first_block = step == 0;
    const bool need_mask = key_end - key0 < kTile || pos_max(PosDesc32{start0, a.kpos.len0, start1, a.kpos.len1}, key0, key_end) > qmin;
    if (!Op::kAhead) op.load_k(a.k, tile, lane);
    op.stash_k(lds, lane);
    if (!Op::kAhead) op.load_v(a.v, tile, lane);
    turn += kWaves;
    more = next_tile();
    tile = tile_now(more);
    if (Op::kAhead) op.load_k(a.k, tile, lane);
    typename Op::Scores s = op.scores(lds, q_lds, lane);
    if (sizeof(T) == 2) op.load_v(a.v, tile, lane);   // (V has gone to LDS)
    if (need_mask) {
      // key key0 + first_key() + c (c known at compile time) is visible if c does not exceed this row's bound in the run
      // that the key belongs to; worked out here, from a lane index the compiler cannot see through, and not kept
      int t = lane;
      asm volatile("" : "+v"(t));
      const int first = key0 + Op::first_key(t);
      const int qp = a.causal ? pos_of(qpos, min(row0 + Op::row_of(t), a.Lq - 1)) : kNever;
      const int in_run0 = a.kpos.len0 - first;
      const int bound0 = min(qp - start0, key_end - 1) - first, bound1 = min(qp - start1, key_end - 1 - a.kpos.len0) + in_run0;
#pragma unroll
      for (int e = 0; e < Op::kScores; ++e) {
        const int c = Op::key_step(e);
        s[e] = c <= (c < in_run0 ? bound0 : bound1) ? s[e] : -INFINITY;
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < Op::kScores; ++e) mx = fmaxf(mx, s[e]);
    mx = Op::max_of_row(mx);
    if (!shared_first) {
      int t = lane;   // places in LDS derived here, from a lane index the compiler cannot see through: kept, they are spilled
      asm volatile("" : "+v"(t));
      if (wave < 2 && t < 32) first_s[wave][t] = (wave == 0 || first_block) ? mx : -INFINITY;
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
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < (int)(sizeof(o[0]) / 4); ++e) o[nb][e] *= alpha;
      m = m_new;
    }
    const float mc = m == -INFINITY ? 0.f : m * a.scale_log2;
#pragma unroll
    for (int e = 0; e < Op::kScores; ++e) {
      s[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], a.scale_log2, -mc));
      l += s[e];
    }
    op.accumulate(s, o, lds, lane);
    if (Op::kAhead && sizeof(T) == 4) op.load_v(a.v, tile, lane);
  }
  if (!shared_first) {   // no tile for this wave
    if (wave < 2 && lane < 32) first_s[wave][lane] = -INFINITY;
    __syncthreads();
  }

  // ---- the waves' states are combined: common maximum, scaled outputs side by side in LDS, summed row by row
  int end_lane = lane;   // (a lane index of its own for the epilogue: what derives from it is not kept across the loop)
  asm volatile("" : "+v"(end_lane));
  constexpr int PER_ROW = HS / 4, ROWS_PER_PASS = kWaves * 64 / PER_ROW, PASSES = (kRows + ROWS_PER_PASS - 1) / ROWS_PER_PASS;
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
  const int end_row = Op::row_of(end_lane);
  l = Op::sum_of_row(l);
  if (end_lane < kRows) {
    m_s[wave][end_row] = m;
    l_s[wave][end_row] = l;
  }
  __syncthreads();
  // (every loop over the waves is unrolled, all its LDS reads in flight at once: a wave that had no tile adds zeros)
  float mw[kWaves], m_all = -INFINITY;
#pragma unroll
  for (int j = 0; j < kWaves; ++j) mw[j] = m_s[j][end_row];
#pragma unroll
  for (int j = 0; j < kWaves; ++j) m_all = fmaxf(m_all, mw[j]);
  if constexpr (STATE) m_all = fmaxf(m_all, m_state_s[end_lane & 31]);
  const float mc = m_all == -INFINITY ? 0.f : m_all * a.scale_log2;
  {
    const float f = __builtin_amdgcn_exp2f(m * a.scale_log2 - mc);
    float* dst = (float*)smem + (wave * kRows + end_row) * OSTR;
#pragma unroll
    for (int gi = 0; gi < Op::kGroups; ++gi) *(f32x4*)(dst + Op::group_dim(gi, end_lane)) = Op::group(o, gi) * f;
  }
  if (wave == 0 && (STATE || end_lane < kRows)) {
    float tot = 0.f;
#pragma unroll
    for (int j = 0; j < kWaves; ++j) tot += l_s[j][end_row] * __builtin_amdgcn_exp2f(mw[j] * a.scale_log2 - mc);
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
      inv_s[end_row] = tot > 0.f ? 1.f / tot : 0.f;   // a row that saw no key: O = 0, LSE = -inf
      if (row0 + end_row < a.Lq)
        a.lse[(((int64_t)rank * a.bs + b) * a.hq + h) * a.Lq + row0 + end_row] = tot > 0.f ? m_all * a.scale + logf(tot) : -INFINITY;
    }
  }
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    const int rr = pass * ROWS_PER_PASS + (int)threadIdx.x / PER_ROW, c = (int)threadIdx.x % PER_ROW;
    if (kRows % ROWS_PER_PASS && rr >= kRows) break;
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
      OutT* dst = (OutT*)a.o + q_row(row0 + rr) + 4 * c;
      if constexpr (sizeof(OutT) == 4) *(f32x4_any*)dst = sum;
      else *(u32x2_any*)dst = u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
    }
  }
}

template <typename T, int HS, typename OutT, bool STATE = false, int ROWS = 32, int CROSS = kNoCross>
int launch_typed(WsArgs a, int64_t grid, hipStream_t stream) {
  constexpr size_t lds = lds_bytes<T, HS, ROWS>();
  auto kern = wave_split_attn_fwd<T, HS, OutT, STATE, ROWS, CROSS>;
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

// (a whole forward of several shards: its results are of the inputs' type)
template <int CROSS>
int launch_crossing(const WsArgs& a, int hs, int in_dtype, int rows, int64_t grid, hipStream_t stream) {
  if (in_dtype == USP_FP32 && rows == 16)
    return hs == 128 ? launch_typed<float, 128, float, false, 16, CROSS>(a, grid, stream) : launch_typed<float, 64, float, false, 16, CROSS>(a, grid, stream);
  if (in_dtype == USP_FP32)
    return hs == 128 ? launch_typed<float, 128, float, false, 32, CROSS>(a, grid, stream) : launch_typed<float, 64, float, false, 32, CROSS>(a, grid, stream);
  return hs == 128 ? launch_typed<__bf16, 128, __bf16, false, 32, CROSS>(a, grid, stream) : launch_typed<__bf16, 64, __bf16, false, 32, CROSS>(a, grid, stream);
}

int launch(WsArgs a, const FastDiv& n_k, int hs, int in_dtype, int o_dtype, hipStream_t stream) {
  a.g = a.hq / a.hkv;
  a.by_hkv = fast_div(a.hkv); a.by_bs = fast_div(a.bs); a.by_ranks = fast_div(a.n_ranks);
  a.by_g = fast_div(a.g); a.by_U = fast_div(a.U);
  const int64_t heads = (int64_t)a.hq * a.bs * a.n_ranks;
  const int rows = in_dtype == USP_FP32 ? wave_split_fp32_rows(a.Lq, heads, (int64_t)a.R * ((a.Lk + kTile - 1) / kTile), a.causal) : 32;
  a.n_qtiles = (a.Lq + rows - 1) / rows;
  auto strides = [&](int heads, const FastDiv& n, uint64_t& ring, uint64_t& run, uint64_t& jump) {
    run = (uint64_t)n.d * heads * hs;
    ring = run * a.bs * a.U;
    jump = run * (a.bs - 1);
  };
  strides(a.q_heads, a.n_q, a.q_ring, a.q_run, a.q_jump);
  strides(a.kv_heads, n_k, a.kv_ring, a.kv_run, a.kv_jump);
  const Cross cross = wave_split_crossing(n_k.d, a.U, a.R, a.bs, (int64_t)a.kv_heads * hs * dtype_size(in_dtype), in_dtype, hs, rows);
  a.tiles.one = a.kv_jump == 0 || cross != kNoCross;
  a.tiles.by_n = n_k;
  a.tiles.by_tiles = fast_div((n_k.d + kTile - 1) / kTile);
  if (!a.causal) a.kpos = BlockPositions{0, 0, a.Lk, 0, 0, 0};
  a.scale_log2 = a.scale * 1.4426950408889634f;
  const int64_t grid = (int64_t)a.n_qtiles * heads;
  if (grid > 0x7fffffffll) return USP_ERR_UNSUPPORTED;
  if (a.state) {   // bf16 data
    if (hs == 128) return o_dtype == USP_FP32 ? launch_typed<__bf16, 128, float, true>(a, grid, stream) : launch_typed<__bf16, 128, __bf16, true>(a, grid, stream);
    return o_dtype == USP_FP32 ? launch_typed<__bf16, 64, float, true>(a, grid, stream) : launch_typed<__bf16, 64, __bf16, true>(a, grid, stream);
  }
  if (cross == kOneCross) return launch_crossing<kOneCross>(a, hs, in_dtype, rows, grid, stream);
  if (cross == kAnyCross) return launch_crossing<kAnyCross>(a, hs, in_dtype, rows, grid, stream);
  if (in_dtype == USP_FP32 && rows == 16) {
    if (hs == 128) return o_dtype == USP_FP32 ? launch_typed<float, 128, float, false, 16>(a, grid, stream) : launch_typed<float, 128, __bf16, false, 16>(a, grid, stream);
    return o_dtype == USP_FP32 ? launch_typed<float, 64, float, false, 16>(a, grid, stream) : launch_typed<float, 64, __bf16, false, 16>(a, grid, stream);
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
  a.n_q = fast_div(p.L / ((int64_t)p.ulysses * p.ring));
  a.Lq = a.Lk = (int)(p.L / p.ring);
  a.causal = p.causal ? 1 : 0;
  const int c = a.Lq / 2;
  a.qpos = a.kpos = p.split == USP_SPLIT_ZIGZAG ? BlockPositions{0, c, c, (2 * p.ring - 1) * c, c, c} : BlockPositions{0, a.Lq, a.Lq, 0, 0, 0};
  a.scale = scale;
  return launch(a, a.n_q, p.hs, p.dtype, p.dtype, stream);
}

int launch_wave_split_block_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int bs, int64_t Lq,
                                int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc& qpos,
                                const usp_posdesc& kpos, int in_dtype, int o_dtype, hipStream_t stream, const RingState* state) {
  WsArgs a = {};
  a.q = q; a.k = k; a.v = v; a.o = o; a.lse = lse;
  a.bs = bs; a.hq = a.q_heads = hq; a.hkv = a.kv_heads = hkv;
  a.U = a.R = a.n_ranks = 1;
  a.Lq = (int)Lq; a.n_q = fast_div(Lq);
  a.Lk = (int)Lk;
  a.causal = causal;
  if (state) {
    a.state = state->state; a.state_first = state->first; a.state_last = state->last;
    a.state_records = (int)((Lq + 255) / 256) * 8;
  }
  a.qpos = BlockPositions{(int)qpos.start0, 0, (int)qpos.len0, (int)qpos.start1, 0, (int)qpos.len1};
  a.kpos = BlockPositions{(int)kpos.start0, 0, (int)kpos.len0, (int)kpos.start1, 0, (int)kpos.len1};
  a.scale = scale;
  return launch(a, fast_div(Lk), hs, in_dtype, o_dtype, stream);
}

}  // namespace usp
