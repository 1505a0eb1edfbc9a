// Blockwise attention (Sec. 2: SP-Ring's blockwise loop; Eq. 1 restricted to the K/V blocks given):
// S = scale * Q K^T -> position mask -> online softmax over key tiles -> P V, returning O (the partial O of
// one ring step, or the final O when the launch covers the whole ring loop) and the per-row log-sum-exp.
//
// gfx950 design (bf16 instance)
//   * MFMA v_mfma_f32_32x32x16_bf16, fp32 accumulation.  The score tile is computed TRANSPOSED,
//     S^T = K Q^T: a lane then owns one query column (lane % 32) and 16 keys per 32-key block in
//     its accumulator registers, so the softmax row max / row sum are in-register reductions plus
//     one exchange between lanes l and l^32.  The accumulator layout of S^T is also the B-operand
//     layout of the second product O^T = V^T P^T (same lane <-> query, 8 keys per 16-key step), so
//     P never leaves registers.
//   * A workgroup owns BM = NWAVES * NQB * 32 query rows of one (batch, head); Q fragments stay in
//     registers for the whole kernel.  K and V tiles of KT keys are staged in LDS, double
//     buffered, fetched to registers one tile ahead while the current tile is being multiplied.
//   * K is read from LDS as row-major 16 B fragments (A operand, rows = keys).  V stays row-major
//     in LDS too; the V^T A-operand (rows = head dims, k = keys) is produced by the LDS transpose
//     read ds_read_b64_tr_b16, which hands each lane 4 consecutive keys of its head dim.
//   * exp2 with log2(e) folded into the scale; masks only on tiles that straddle the causal
//     boundary or the ragged tail; key tiles that are invisible to the whole query tile are
//     never loaded; the O accumulator is rescaled only when some row maximum moved.
//   * One workgroup per CU, persistent: work items (query tile x head x batch) are drawn from
//     counters in device memory, heaviest query tiles first (descending local index under a
//     causal mask), KV group fastest; a workgroup prefers the items whose KV heads its XCD's L2
//     already serves (attn_device.h).  K/V tiles are fetched through buffer descriptors.
#include <algorithm>
#include <numeric>
#include <type_traits>

#include "attn_device.h"
#include "usp_internal.h"

namespace usp {
namespace {

using namespace dev;

constexpr int kMaxBlocks = USP_MAX_RING_BLOCKS;

// One launch covers n_blocks K/V blocks of Lk keys each (the ring steps of one rank, Algorithm 1 step 5): the
// online-softmax state of a query row stays in registers from the first block to the last, so no partial results
// and no merge pass exist.  n_blocks = 1 is the plain single ring step.
struct AttnArgs {
  const void* q;
  const void* k[kMaxBlocks];
  const void* v[kMaxBlocks];
  void* o;
  float* lse;
  int bs, hq, hkv, g;
  int Lq, Lk;
  int n_qtiles;
  int tiles_run0;     // > 0: the query tiles of the first run of positions, the others begin at row qpos.len0 (RowTiles)
  int n_blocks;
  int causal;
  float scale;        // natural-units scale (for the LSE)
  float scale_log2;   // scale * log2(e)
  PosDesc32 qpos;
  PosDesc32 kpos[kMaxBlocks];
  // Where Q rows are read and O rows written.  seq_n == 0: dense [bs,Lq,hq,hs] (the layout after the forward
  // all-to-all).  seq_n > 0: straight from / to the sequence-layout shards of the rank's Ulysses group,
  // [U][bs][seq_n][seq_heads][hs] with this rank's heads at seq_head0: the all-to-all of Q (Algorithm 1 step 2)
  // and of O (step 6) folded into the one read of Q and the one write of O that the kernel does anyway.
  int seq_n, seq_heads, seq_head0;
  // Heads in a row of K and of row-major V: hkv (dense), or all KV heads of the model where the kernel reads a batch
  // of one straight from the sequence-layout shards of the rank's Ulysses group (k and v then point at the rank's first
  // head).  The staged copy this replaces was a launch ahead of every forward, 5.6 us at L = 8192.
  int kv_pitch;
  int ticket_slot;   // counter the workgroups draw their work items from (MFMA kernel)
  int n_items;       // work items of the launch: query tiles x heads x batch
  int n_queues;      // gcd(8, batch x KV heads): item w waits in queue w mod n_queues
  // Key split (launch_attn_fwd_partials): an item is (query tile, head, batch, ONE block), the blocks may differ in
  // their number of keys, and the item's O (fp32, dense) and LSE go to the block's own partial result.  Otherwise
  // (per_block = 0) an item walks all blocks, every block holds Lk keys and the result goes to o / lse.
  int per_block;
  // Mixed launch (launch_attn_fwd_mixed, kernel instance MIXED): the first n_split_items items are (query tile, head,
  // batch, ONE block) items as above, over the n_split_tiles query tiles that come first in item order (the heaviest
  // under a causal mask), each with its partial result; the items after them are whole items over the other query
  // tiles, which walk all blocks and write o / lse.  Every block holds lk_blk[j] keys.
  int n_split_items, n_split_tiles;
  int lk_blk[kMaxBlocks];
  void* o_part[kMaxBlocks];
  float* lse_part[kMaxBlocks];
  int part_row0[kMaxBlocks];   // a partial result holds the rows from here on (of every batch entry)
  // Running state of a ring that delivers its blocks one per call (launch_block_attn_fwd_state): the online-softmax
  // state of every query row (running maximum m, sum l, unnormalised O^T accumulator) in the kernel's own register
  // layout, one record of state_record_floats() per 32-row block of a (batch, head): read at the start of an item
  // unless state_first, written at its end instead of O and LSE unless state_last.  Null: no state (all other paths).
  float* state;
  int state_first, state_last;
};

// The arguments of a launch whose items are listed.  Instance STATE: the query tiles that its middle steps walk.  Instance
// MIXED: a tile and the piece of the keys (listed_item()), heaviest first, every entry once per head and batch entry.
struct ListedArgs : AttnArgs {
  int n_listed;                         // 0: every tile, in the usual order
  uint32_t list[kMaxListedItems / 2];   // two to a word
};

// floats of one 32-row state record: the O^T accumulator (hs / 32 x 16 registers x 64 lanes), then m and l per lane
constexpr size_t state_record_floats(int hs) { return (size_t)(hs / 32) * 16 * 64 + 2 * 64; }

// The scalar arguments as one work item of the MFMA kernel sees them (read anew for every item, see the kernel).
struct ItemArgs {
  const void* q;
  void* o;
  float* lse;
  int bs, hq, hkv, g;
  int Lq, Lk;
  int n_qtiles;
  int n_blocks;
  int causal;
  float scale, scale_log2;
  PosDesc32 qpos;
  int seq_n, seq_heads, seq_head0;
  int kv_pitch;
};

// element offset of (batch b, local row, local head h) in the Q / O tensor
template <typename Args>
__device__ inline size_t qo_offset(const Args& a, int b, int row, int h, int hs) {
  if (a.seq_n == 0) return (((size_t)b * a.Lq + row) * a.hq + h) * hs;
  const int shard = row / a.seq_n, s = row - shard * a.seq_n;
  return ((((size_t)shard * a.bs + b) * a.seq_n + s) * a.seq_heads + a.seq_head0 + h) * hs;
}

// -------------------------------------------------------------------------------------------
// bf16 MFMA kernel, software pipelined: while the softmax of key tile j runs on the vector ALU,
// the matrix core already computes the scores of tile j+1, then P(j) V(j) (TRAILING: P(j) V(j) a tile later).
// -------------------------------------------------------------------------------------------
// VT: the V blocks come in key-tile-transposed layout (usp.h: USP_SEQ_TO_HEAD_VT): per (batch, KV head) tiles of 64
// keys stored [hs][64 keys], the keys of each group of 16 in the order 0-3, 8-11, 4-7, 12-15.  The A operand of
// O^T = V^T P^T (rows = head dims, 8 keys per lane) is then ONE 16-byte row read per product instead of two LDS
// transpose reads: 32 LDS reads per step and wave (the minimum: one fragment per product) instead of 48, and the
// LDS pipe, which issues a read every ~7 cycles whatever its width, was the busiest unit of the kernel.
template <int HS, int NQB, int NWAVES, int KT, int WPE, typename OutT, bool STATE = false, bool VT = false, bool MIXED = false, bool TRAILING = false>
__global__ __attribute__((amdgpu_flat_work_group_size(NWAVES * 64, NWAVES * 64), amdgpu_waves_per_eu(WPE, WPE)))
void block_attn_fwd_mfma(const std::conditional_t<STATE || MIXED, ListedArgs, AttnArgs>) {
  using Args = std::conditional_t<STATE || MIXED, ListedArgs, AttnArgs>;
  static_assert(!STATE || NQB == 1, "the state record is laid out for one 32-row block per wave");
  static_assert(!MIXED || (!STATE && sizeof(OutT) == 2), "the mixed launch writes bf16 results and fp32 partials");
  static_assert(!VT || KT == 64, "the transposed V layout is made of 64-key tiles");
  constexpr int NT = NWAVES * 64;
  constexpr int BM = NWAVES * NQB * 32;
  constexpr int KSTEPS = HS / 16;          // MFMA k-steps of Q K^T
  constexpr int DB = HS / 32;              // 32-wide head-dim blocks of O^T
  constexpr int KB = KT / 32;              // 32-key blocks of S^T
  constexpr int PS = KT / 16;              // MFMA k-steps of P V
  constexpr int KSTR = HS * 2 + 48;        // LDS row stride of K in bytes: an odd number of 16 B chunks, no bank conflicts on the row reads
  // V rows: an odd multiple of 64 B, no bank conflicts on the transpose reads; transposed tiles: rows of KT keys
  // (128 B) padded to an odd number of 16 B chunks like the K rows
  constexpr int VSTR = VT ? KT * 2 + 16 : HS * 2 + 64;
  constexpr int KBYTES = KT * KSTR, VBYTES = VT ? HS * VSTR : KT * VSTR;
  constexpr int VT_TILE_BYTES = HS * KT * 2;   // one transposed tile in global memory: [HS][KT] bf16, contiguous
  constexpr int CHUNKS = KT * HS / 8;      // 16 B chunks per tile (K and V alike)
  constexpr int CPT = CHUNKS / NT;         // chunks per thread
  // Finished rows leave in whole lines (put_rows).  Only where items are short and many end in fp32 partial results: L = 8192
  // of Ulysses 8 88.1 -> 86.2 us; in the uncut instances, whose items are 100 us and more, nothing was gained (L = 32768 971
  // and 972 us) and the registers that it takes at the end changed the tile loop's (L = 212992 0.5 % slower).
  constexpr bool LINES = MIXED;
  constexpr float kRescaleThreshold = 8.0f;   // in log2 units: P stays below 2^8
  // TRAILING (head size 64, where second_product_trails()): half the products to as many weights, and registers to spare.  The vector
  // ALU is the busier unit (a wave issues an instruction of it every eight cycles at most, two waves one every four), so P V runs a tile behind, under the next tile's
  // weights like that tile's scores, and no row maxima are formed while a tile's weights stay within their bound (their sum,
  // which is formed anyway, tells).  One rank of Ulysses 8, us: L = 32768 601 -> 586, 65536 without a mask 4720 -> 4650, 17776
  // without a mask 371 -> 357; ring 8, 32768 610 -> 598, its eight steps with a state 667 -> 656.  The products spread evenly between the
  // weights' instructions instead of where the compiler leaves them: 5 % slower.  At head size 128, where the products take longer
  // than the weights, it fits the registers and is 1.5 to 4 % slower (L = 32768 963 -> 981, 212992 19990 -> 20770).
  // Row maxima on demand.  A tile whose weights sum up to more than kSumLimit for a lane (a row's first keys: infinity) is formed
  // again with its maxima, and the accumulators are scaled, at the end of the step, where nothing hides it: 900 cycles of a step's
  // 2600 if one of the workgroup's 256 rows asks.  Twice within kMovesApart tiles, and the wave watches: it forms the maxima
  // ahead of the next kWatched tiles' weights, as the other loop does, and lets P V of the tile before finish before it
  // scales.  The other loop / without watching / with it, one rank of Ulysses 8, us: L = 16384, Q times 1 169 / 165 / 165, 10
  // 175 / 194 / 183, 30 170 / 208 / 177, scores that rise by 1000 over the length 174 / 231 / 184; no mask, 17776 393 / 362 / 358,
  // 403 / 405 / 394, 389 / 419 / 383, 407 / 523 / 408.  Watching always costs 5 % (L = 32768 570 -> 601, 17776 349 -> 368).  Limits up to 2^40
  // instead are as fast, but a row's largest weight is then rarely 1, which bf16 has exactly: O was 12 to 20 % further from 64 bits
  // with Q times 4 to 16 (as it is: 5 % nearer to 2 % further than the other loop's, and the same with Q times 1).
  constexpr float kSumLimit = 1024.f;
  constexpr float kWatchedGrowth = 5.f;       // in log2 units: 32 weights of 2^5 are within the limit
  constexpr int kMovesApart = 12, kWatched = 32;
  // No maximum yet: finite, so that a key that is masked has a weight of zero.  With infinity it was NaN, and while a wave had a row
  // that saw nothing every tile was formed twice: ring steps with a state, L = 32848, ring 8, its own block last 1755 us, first 1610; now 1602
  // and 1603.
  constexpr float kNoMaximum = 3.4028235e38f;
  static_assert(!TRAILING || (HS == 64 && NQB == 1), "one 32-row block per wave");
  static_assert(CHUNKS % NT == 0, "tile must split evenly over the workgroup");

  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* const kbuf = smem;                  // [2][KBYTES]
  char* const vbuf = smem + 2 * KBYTES;     // [2][VBYTES]

  // ---- persistent workgroups: one per CU, each draws work items until none is left.  Item order: KV group
  //      fastest, then head within group, then query tile (heavy first).
  // The next item is drawn when the current one reaches its epilogue (not earlier: an item taken long before it is
  // started is no longer the next one in line when it starts, which is what balances the CUs): thread 0 asks at
  // the start of the epilogue and reads the answer after it, so the latency of the draw hides behind the stores
  // of O.  The item's number waits in LDS, two slots in turn: the next number may be written while slower waves
  // still read the current one.
  __shared__ int next_item[2];
  __shared__ unsigned empty_queues;   // thread 0's record of the item queues it has found empty
  int turn = 0;
  if (threadIdx.x == 0) {
    auto ap0 = (const __attribute__((address_space(4))) Args*)__builtin_amdgcn_kernarg_segment_ptr();
    // the first item is given, not drawn
    next_item[0] = ItemQueues{ap0->ticket_slot, ap0->n_items, (int)gridDim.x, ap0->n_queues}.first_item(blockIdx.x);
    empty_queues = 0;
  }
  for (;;) {
    // The kernel arguments are read anew for every item, through a pointer to the argument segment that the
    // compiler cannot see through.  Read once, everything derived from them (reciprocals of the item decode, strides,
    // flags) would be hoisted out of the item loop and held in scalar registers across it; there are not enough,
    // and the overflow goes to lanes of a vector register that the tile loop cannot spare.
    auto ap = (const __attribute__((address_space(4))) Args*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ap));
    const int n_items = ap->n_items;
    // Every item given, none left to draw: no counter is touched.  (Looking for one took 3 to 5 us at the end of a launch.)
    const bool drawing = !STATE || n_items > (int)gridDim.x;
    __syncthreads();   // the previous item is done with LDS, and next_item[turn] has been written
    int w = __builtin_amdgcn_readfirstlane(next_item[turn]);
    turn ^= 1;
    if (w >= n_items) {
      if (drawing && threadIdx.x == 0) ItemQueues{ap->ticket_slot, n_items, (int)gridDim.x, ap->n_queues}.leave();
      break;
    }
    ItemArgs a;
    a.q = ap->q; a.o = ap->o; a.lse = ap->lse;
    a.bs = ap->bs; a.hq = ap->hq; a.hkv = ap->hkv; a.g = ap->g;
    a.Lq = ap->Lq; a.Lk = ap->Lk;
    a.n_qtiles = ap->n_qtiles; a.n_blocks = ap->n_blocks; a.causal = ap->causal;
    a.scale = ap->scale; a.scale_log2 = ap->scale_log2;
    a.qpos = PosDesc32{ap->qpos.start0, ap->qpos.len0, ap->qpos.start1, ap->qpos.len1};
    a.seq_n = ap->seq_n; a.seq_heads = ap->seq_heads; a.seq_head0 = ap->seq_head0; a.kv_pitch = ap->kv_pitch;
    const int n_groups = a.bs * a.hkv;
    // The lane constants are derived anew for every item from a thread index the compiler cannot see through:
    // hoisted out of the item loop they would stay in registers across it, and the tile loop has none to spare.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform by construction: keep what derives from it in scalar registers
    const int l32 = lane & 31, hl = lane >> 5;
    bool per_block = ap->per_block != 0;
    bool listed = false;
    if constexpr (MIXED) {
      listed = ap->n_listed > 0;
      if (!listed) {
        per_block = w < ap->n_split_items;     // the split items come first
        if (!per_block) w -= ap->n_split_items;
      }
    }
    const int group = w % n_groups; w /= n_groups;
    const int hg = w % a.g;
    int t = w / a.g;
    int blk0 = 0, blk1 = a.n_blocks;         // the blocks this item walks
    int entry = 0;
    if constexpr (STATE || MIXED) {
      if (STATE ? ap->n_listed > 0 : listed) entry = (int)((ap->list[t >> 1] >> (16 * (t & 1))) & 0xffffu);
    }
    if (MIXED && listed) {
      const int piece = entry >> kListedTileBits;
      per_block = piece != kListedWhole;
      if (per_block) {
        blk0 = piece;
        blk1 = blk0 + 1;
      }
    } else if (per_block) {
      blk0 = t % a.n_blocks;
      blk1 = blk0 + 1;
      t /= a.n_blocks;
    } else if constexpr (MIXED) {
      t += ap->n_split_tiles;
    }
    // (a mixed launch counts its tiles from the last one down whatever the mask: its cut tiles are the last rows)
    int qtile = (a.causal || MIXED) ? a.n_qtiles - 1 - t : t;
    if constexpr (STATE) qtile = ap->n_listed ? entry : qtile;
    if constexpr (MIXED) qtile = listed ? entry & ((1 << kListedTileBits) - 1) : qtile;
    const int b = group / a.hkv, kvh = group % a.hkv;
    const int h = kvh * a.g + hg;

    int tile_row0 = qtile * BM, row_end = a.Lq;   // rows from row_end on are none of this tile's
    if constexpr (!STATE) {   // (the state's records are 256 rows in a row)
      const int run0 = ap->tiles_run0;
      if (run0 > 0) {
        if (qtile < run0) row_end = a.qpos.len0;
        else tile_row0 = a.qpos.len0 + (qtile - run0) * BM;
      }
    }
    const int tile_row1 = min(row_end, tile_row0 + BM);
    const int wave_row0 = tile_row0 + wave * (NQB * 32);

    if constexpr (STATE) {
      // A middle step of a step-by-step ring in which this query tile sees no key of the block (under the zigzag
      // split half of a rank's rows see nothing of most blocks): the rows' state stays as it is, so it is neither
      // read nor written back, and the item ends here.  (The first step writes the initial state, the last one the
      // output: those walk every item.)
      if (!ap->state_first && !ap->state_last && !ap->n_listed) {
        bool any = false;
        for (int blk = 0; blk < a.n_blocks; ++blk) {
          const PosDesc32 kp = {ap->kpos[blk].start0, ap->kpos[blk].len0, ap->kpos[blk].start1, ap->kpos[blk].len1};
          const TileRanges t = visible_key_tiles<KT>(a.causal, a.qpos, kp, a.Lk, tile_row0, tile_row1);
          any = any || (t.a1 - t.a0) + (t.b1 - t.b0) > 0;
        }
        if (!any) {   // workgroup-uniform
          if (threadIdx.x == 0) {
            const ItemQueues queues = {ap->ticket_slot, n_items, (int)gridDim.x, ap->n_queues};
            unsigned empty = empty_queues;
            next_item[turn] = drawing ? queues.finish(queues.begin(empty), empty) : n_items;
            empty_queues = empty;
          }
          continue;
        }
      }
    }

    const __bf16* qg = (const __bf16*)a.q;
    const size_t kv_head_off = ((size_t)b * a.Lk * a.kv_pitch + kvh) * HS * 2;   // bytes; + key * kv_pitch * HS * 2
    // transposed V: the tiles of (batch, KV head) are contiguous; a.Lk (the batch stride in rows) gives their number
    const size_t vt_head_off = ((size_t)b * a.hkv + kvh) * (size_t)((a.Lk + KT - 1) / KT) * VT_TILE_BYTES;
    int Lk_b = a.Lk;   // keys of the current block (a.Lk stays the batch stride of every block's tensors)

    // ---- Q fragments (B operand of S^T = K Q^T): lane = query l32, dims 16*ks + 8*hl .. +7
    bf16x8 qf[NQB][KSTEPS];
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const int rr = min(wave_row0 + qb * 32 + l32, row_end - 1);
      const __bf16* src = qg + qo_offset(a, b, rr, h, HS) + 8 * hl;
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) qf[qb][ks] = *(const bf16x8*)(src + 16 * ks);
    }

    // per-block state of the tile walk (workgroup-uniform), set at the top of the block loop
    const char* kg = nullptr;
    const char* vg = nullptr;
    PosDesc32 kpos = {0, 0, 0, 0};
    TileRanges tr = {0, 0, 0, 0};
    int na = 0, nt = 0;
    int free_a = 0, free_b0 = 0, free_b1 = 0;   // walk positions [0, free_a) and [free_b0, free_b1): tiles this wave need not mask
    auto tile_of = [&](int it) { return it < na ? tr.a0 + it : tr.b0 + (it - na); };

    f32x16 oacc[NQB][DB];
    float m_run[NQB], l_run[NQB];
    float zero = 0.f;
    asm volatile("" : "+v"(zero));   // not a constant to the compiler: it would share one zeroed register tuple between items
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      m_run[qb] = -INFINITY;
      l_run[qb] = zero;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[qb][db][i] = zero;
    }

    // ---- running state of a step-by-step ring: this wave's record (one per 32-row block of the head)
    // (an instance of its own, STATE: in the plain instance the code below is not there at all)
    float* st_rec = nullptr;
    if constexpr (STATE) {
      float* const st = ap->state;
      {
        st_rec = st + ((((size_t)b * a.hq + h) * a.n_qtiles + qtile) * NWAVES + wave) * state_record_floats(HS);
      }
    }
    // (the first step's loads find an empty range and give zeros: no branch, no second copy of the accumulators)
    auto state_rsrc = [&]() {
      return __builtin_amdgcn_make_buffer_rsrc((void*)st_rec, 0, ap->state_first ? 0 : (int)(state_record_floats(HS) * sizeof(float)), kRawBufferFlags);
    };
    auto load_state_sums = [&]() {   // m (-inf: no state yet) and l
      const __amdgpu_buffer_rsrc_t rec = state_rsrc();
      const uint32_t m = __builtin_amdgcn_raw_buffer_load_b32(rec, lane * 4, DB * 4096, 0);
      const uint32_t l = __builtin_amdgcn_raw_buffer_load_b32(rec, lane * 4, DB * 4096 + 256, 0);
      m_run[0] = ap->state_first ? -INFINITY : __builtin_bit_cast(float, m);
      l_run[0] = __builtin_bit_cast(float, l);
    };
    auto load_state_acc = [&]() {
      const __amdgpu_buffer_rsrc_t rec = state_rsrc();
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const u32x4 v4 = __builtin_amdgcn_raw_buffer_load_b128(rec, lane * 16, (db * 4 + j) * 1024, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t x = v4[e];
            oacc[0][db][4 * j + e] = __builtin_bit_cast(float, x);
          }
        }
    };

    // TRAILING
    float neg_mc = kNoMaximum;                     // -m in the exponent's units
    float late_alpha = 1.f;                        // the accumulators' factor for the maximum's last move,
    bool late = false;                             // still to come, behind the products of the tile before
    int last_move = -kMovesApart, watched = 0;     // the tile of the last move; tiles still to be watched

    // wave-level bounds for the mask decision
    const int wave_row1 = min(row_end, wave_row0 + NQB * 32);
    const bool wave_live = wave_row0 < row_end;
    const int wave_qmin = (a.causal && wave_live) ? pos_min(a.qpos, wave_row0, wave_row1) : 0;

    // ---- staging: each thread moves CPT 16 B chunks of a K tile and of a V tile
    const int st_row = tid / (HS / 8), st_col = tid % (HS / 8);
    constexpr int ROWS_PER_PASS = NT / (HS / 8);
    u32x4 kreg[CPT], vreg[CPT];
    // Tiles are read through a buffer descriptor built per tile in scalar registers: base = the tile's first row
    // (this KV head), extent = up to the end of its last valid row.  Each thread adds a 32-bit byte offset that is
    // the same for every tile; rows past the last key (ragged final tile only) lie beyond the extent and read as
    // zeros (the mask hides those keys).  No 64-bit address arithmetic on the vector ALU, no clamping.
    const uint32_t row_bytes = (uint32_t)a.kv_pitch * HS * 2;
    uint32_t st_off[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) st_off[c] = (uint32_t)(st_row + c * ROWS_PER_PASS) * row_bytes + st_col * 16;
    // (`tile` is the tile's number in the block, not its place in the walk; the extent is one of two values that
    // are worked out once per block: a full tile's, or that of the block's ragged last tile)
    int full_tiles = 0, full_extent = 0, ragged_extent = 0;
    auto fetch = [&](const char* base, int tile, u32x4* reg) {
      const char* tb = base + (uint64_t)((uint32_t)tile * KT) * row_bytes;
      const __amdgpu_buffer_rsrc_t tile_rsrc = __builtin_amdgcn_make_buffer_rsrc(
          (void*)tb, 0, tile < full_tiles ? full_extent : ragged_extent, kRawBufferFlags);
#pragma unroll
      for (int c = 0; c < CPT; ++c) reg[c] = __builtin_amdgcn_raw_buffer_load_b128(tile_rsrc, (int)st_off[c], 0, 0);
    };
    auto stash = [&](char* buf, int stride, const u32x4* reg) {
#pragma unroll
      for (int c = 0; c < CPT; ++c) *(u32x4*)(buf + (st_row + c * ROWS_PER_PASS) * stride + st_col * 16) = reg[c];
    };
    // transposed V tiles: 16 KiB (8 KiB at head size 64) contiguous in global memory, chunk c of the tile goes to
    // row c / 8 (a head dim), 16 B column c % 8 of the LDS tile
    auto fetch_vt = [&](const char* base, int tile, u32x4* reg) {
      const char* tb = base + (uint64_t)(uint32_t)tile * VT_TILE_BYTES;
      const __amdgpu_buffer_rsrc_t tile_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)tb, 0, VT_TILE_BYTES, kRawBufferFlags);
#pragma unroll
      for (int c = 0; c < CPT; ++c) reg[c] = __builtin_amdgcn_raw_buffer_load_b128(tile_rsrc, (tid + c * NT) * 16, 0, 0);
    };
    auto stash_vt = [&](char* buf, const u32x4* reg) {
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const int ch = tid + c * NT;
        *(u32x4*)(buf + (ch >> 3) * VSTR + (ch & 7) * 16) = reg[c];
      }
    };
    auto fetch_v = [&](const char* base, int tile, u32x4* reg) {
      if constexpr (VT) fetch_vt(base, tile, reg); else fetch(base, tile, reg);
    };
    auto stash_v = [&](char* buf, const u32x4* reg) {
      if constexpr (VT) stash_vt(buf, reg); else stash(buf, VSTR, reg);
    };

    // ---- S^T = K Q^T for the tile in K buffer kb_ (rows = keys, cols = queries)
    auto qk = [&](const char* kb_, f32x16 (&sacc)[NQB][KB]) {
      const char* krow = kb_ + l32 * KSTR + hl * 16;
      // k-step outermost: consecutive MFMAs go to different accumulators (no back-to-back dependence)
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) {
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk) {
          const bf16x8 kf = *(const bf16x8*)(krow + kbk * 32 * KSTR + ks * 32);
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) {
            if (ks == 0) {
              f32x16 z;
#pragma unroll
              for (int i = 0; i < 16; ++i) z[i] = 0.f;
              sacc[qb][kbk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[qb][ks], z, 0, 0, 0);
            } else {
              sacc[qb][kbk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[qb][ks], sacc[qb][kbk], 0, 0, 0);
            }
          }
        }
      }
    };

    // One pipeline step on tile `it` whose scores are in s_cur.  Unless LAST, the scores of tile it+1
    // are produced into s_next while the softmax of s_cur runs.
    int v_tile = 0;   // number of the V tile the next step prefetches (workgroup-uniform)
    const int grp = lane >> 4, j16 = lane & 15;
    const int v_lane_off = (4 * hl + (j16 >> 2)) * VSTR + (16 * (grp & 1) + 4 * (j16 & 3)) * 2;
    auto step = [&](auto steady_tag, int it, f32x16 (&s_cur)[NQB][KB], f32x16 (&s_next)[NQB][KB]) {
      // steady state (tag true): a next tile and a tile after that exist, no branches in the main block;
      // otherwise the two conditions are evaluated at run time (the last up-to-three tiles)
      constexpr bool STEADY = decltype(steady_tag)::value;
      const bool has1 = STEADY || it + 1 < nt;
      const bool has2 = STEADY || it + 2 < nt;
      const int key0 = tile_of(it) * KT;

      // ---- mask (wave-uniform decision): ragged key tail, or a key of the tile may exceed a query of the wave;
      //      the tiles that need none come in two runs of the walk, worked out once per block
      const bool need_mask = !(it < free_a || (it >= free_b0 && it < free_b1));
      if (need_mask) {
        int qp[NQB];   // the lane's query position: derived here, where it is rarely needed, rather than kept in a register
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) qp[qb] = a.causal ? pos_of(a.qpos, min(wave_row0 + qb * 32 + l32, row_end - 1)) : 0;
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int key = key0 + kbk * 32 + 8 * (i >> 2) + 4 * hl + (i & 3);
            const bool inb = key < Lk_b;
            const int kp = a.causal ? pos_of(kpos, key) : 0;
#pragma unroll
            for (int qb = 0; qb < NQB; ++qb) {
              const bool vis = inb && (!a.causal || kp <= qp[qb]);
              s_cur[qb][kbk][i] = vis ? s_cur[qb][kbk][i] : -INFINITY;
            }
          }
      }

      // ---- row maxima; the running maximum only moves when a row grew by more than the threshold, so the
      //      accumulator rescale is rare (P is then bounded by 2^threshold instead of 1)
      float mc[NQB];
      bool grow = false;
      float mx[NQB];
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        float x = -INFINITY;
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
          for (int i = 0; i < 16; ++i) x = fmaxf(x, s_cur[qb][kbk][i]);
        x = both_halves_max(x);
        mx[qb] = x;
        // first visible key of a row (m_run = -inf) always takes the branch: inf > threshold
        grow = grow || ((x - m_run[qb]) * a.scale_log2 > kRescaleThreshold);
      }
      if (__any(grow)) {
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          const float m_new = fmaxf(m_run[qb], mx[qb]);
          const float mcn = (m_new == -INFINITY) ? 0.f : m_new * a.scale_log2;
          const float alpha = __builtin_amdgcn_exp2f(m_run[qb] * a.scale_log2 - mcn);   // m_run = -inf -> 0
          m_run[qb] = m_new;
          l_run[qb] *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[qb][db][i] *= alpha;
        }
      }
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) mc[qb] = (m_run[qb] == -INFINITY) ? 0.f : m_run[qb] * a.scale_log2;

      // ---- global prefetch: K two tiles ahead, V one tile ahead
      //      (the V tile wanted now is the K tile of the step before: its number is carried over)
      const int k_tile = tile_of(it + 2);
      if (has2) fetch(kg, k_tile, kreg);
      if (has1) fetch_v(vg, v_tile, vreg);
      v_tile = k_tile;
      // keep the loads up here: left alone, the scheduler sinks them to just before the LDS stores below to
      // save registers, and every step then waits out a full global-memory latency
      __builtin_amdgcn_sched_barrier(0);

      // ---- main block: scores of the next tile on the matrix core, softmax of this tile on the vector ALU
      if (has1) qk(kbuf + ((it + 1) & 1) * KBYTES, s_next);

      bf16x8 pf[NQB][PS];
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        float rs = l_run[qb];
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk) {
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            u32x4 pk;
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
              const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[qb][kbk][half * 8 + 2 * pr], a.scale_log2, -mc[qb]));
              const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[qb][kbk][half * 8 + 2 * pr + 1], a.scale_log2, -mc[qb]));
              f32x2 pp = {p0, p1};
              const bf16x2 pb = __builtin_convertvector(pp, bf16x2);
              rs += p0 + p1;
              pk[pr] = __builtin_bit_cast(uint32_t, pb);
            }
            pf[qb][kbk * 2 + half] = __builtin_bit_cast(bf16x8, pk);
          }
        }
        l_run[qb] = rs;
      }

      // ---- O^T += V^T P^T   (rows = head dims, cols = queries, k = keys)
      // MFMA k index e of lane half hl in step s is key 16 s + 8 (e / 4) + 4 hl + (e % 4): the
      // accumulator layout of S^T.  The transpose read returns, for a 16-lane group whose lane j
      // points at (key base + j / 4, dim base + 4 (j % 4)), the 4 keys of dim base + j to lane j.
      const char* vlane = vbuf + (it & 1) * VBYTES + v_lane_off;
#pragma unroll
      for (int s = 0; s < PS; ++s) {
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          bf16x8 vf;
          if constexpr (VT) {
            // row = head dim 32 db + l32, 16 bytes = the lane half's 8 keys of k-step s in the operand's order
            vf = *(const bf16x8*)(vbuf + (it & 1) * VBYTES + (db * 32 + l32) * VSTR + 32 * s + 16 * hl);
          } else {
            const char* p0 = vlane + (16 * s) * VSTR + db * 64;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0 + 8 * VSTR));
            vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
          }
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb)
            oacc[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[qb][s], oacc[qb][db], 0, 0, 0);
        }
      }

      // ---- hand the prefetched tiles to LDS: K(it+2) replaces K(it), V(it+1) replaces V(it-1)
      if (has2) stash(kbuf + (it & 1) * KBYTES, KSTR, kreg);
      if (has1) stash_v(vbuf + ((it + 1) & 1) * VBYTES, vreg);
      __syncthreads();
    };

    // ---- TRAILING: one step on tile `it`, whose scores are in s_cur; the scores of tile it + 1 go to s_next, P(it - 1) V(it - 1)
    //      to the accumulators, P(it) to p_cur
    auto products_v = [&](int it, const bf16x8 (&p)[PS]) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < PS; ++s)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          bf16x8 vf;
          if constexpr (VT) {
            vf = *(const bf16x8*)(vbuf + (it & 1) * VBYTES + (db * 32 + l32) * VSTR + 32 * s + 16 * hl);
          } else {
            const char* p0 = vbuf + (it & 1) * VBYTES + v_lane_off + (16 * s) * VSTR + db * 64;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0 + 8 * VSTR));
            vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
          }
          oacc[0][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, p[s], oacc[0][db], 0, 0, 0);
        }
    };
    auto scale_late = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[0][db][i] *= late_alpha;
      late = false;
    };
    auto largest = [&](const f32x16 (&s)[NQB][KB]) __attribute__((always_inline)) {
      float x = -INFINITY;
#pragma unroll
      for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
        for (int i = 0; i < 16; ++i) x = fmaxf(x, s[0][kbk][i]);
      return both_halves_max(x);
    };
    auto move_maximum = [&](float x) __attribute__((always_inline)) {
#pragma clang fp contract(off)   // (a row whose maximum stays is scaled by one, exactly)
      const float m_new = fmaxf(m_run[0], x);
      const float mcn = (m_new == -INFINITY) ? 0.f : m_new * a.scale_log2;
      late_alpha = __builtin_amdgcn_exp2f(-neg_mc - mcn);   // no maximum yet: 0
      m_run[0] = m_new;
      neg_mc = (m_new == -INFINITY) ? kNoMaximum : -mcn;
      l_run[0] *= late_alpha;
    };
    auto trailing_step = [&](auto steady_tag, int it, f32x16 (&s_cur)[NQB][KB], f32x16 (&s_next)[NQB][KB], const bf16x8 (&p_prev)[PS],
                             bf16x8 (&p_cur)[PS]) __attribute__((always_inline)) {
      constexpr bool STEADY = decltype(steady_tag)::value;   // a tile before, a next one and one after that exist
      const bool has1 = STEADY || it + 1 < nt;
      const bool has2 = STEADY || it + 2 < nt;
      const bool need_mask = !(it < free_a || (it >= free_b0 && it < free_b1));
      if (need_mask | (watched > 0)) {
        if (need_mask) {
          const int key0 = tile_of(it) * KT;
          const int qp = a.causal ? pos_of(a.qpos, min(wave_row0 + l32, row_end - 1)) : 0;
#pragma unroll
          for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int key = key0 + kbk * 32 + 8 * (i >> 2) + 4 * hl + (i & 3);
              const int kp = a.causal ? pos_of(kpos, key) : 0;
              const bool vis = key < Lk_b && (!a.causal || kp <= qp);
              s_cur[0][kbk][i] = vis ? s_cur[0][kbk][i] : -INFINITY;
            }
        }
        if (watched > 0) {
          --watched;
          if (late) scale_late();   // (P(it - 2) V(it - 2) is in; a wave that is late is watched)
          const float x = largest(s_cur);
          if (__any((x - m_run[0]) * a.scale_log2 > kWatchedGrowth)) {   // (a row's first keys: infinity)
            move_maximum(x);
            late = true;
            watched = kWatched;
          }
        }
      }
      if (has2) fetch(kg, tile_of(it + 2), kreg);
      fetch_v(vg, tile_of(it), vreg);
      __builtin_amdgcn_sched_barrier(0);   // (as in step)

      if (has1) qk(kbuf + ((it + 1) & 1) * KBYTES, s_next);
      if (STEADY || it > 0) products_v(it - 1, p_prev);
      auto weights = [&](float n) __attribute__((always_inline)) {
        float sum = 0.f;
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk)
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            u32x4 pk;
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
              const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[0][kbk][half * 8 + 2 * pr], a.scale_log2, n));
              const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[0][kbk][half * 8 + 2 * pr + 1], a.scale_log2, n));
              sum += p0 + p1;
              pk[pr] = pack_bf16(p0, p1);
            }
            p_cur[kbk * 2 + half] = __builtin_bit_cast(bf16x8, pk);
          }
        return sum;
      };
      float sum = weights(neg_mc);
      if constexpr (STEADY) {
        // The eight reads of K ahead of the products, then four and four of V's: left alone, ten come in one burst of all eight
        // waves, behind the barrier.  V in transposed tiles has eight, one for a product; V as rows has sixteen, of which the
        // groups name eight and leave the others where the compiler puts them.  1 to 1.5 % (V as rows, the lengths above, us: 562 -> 557,
        // 4328 -> 4262, 344.5 -> 339.5, 573 -> 569, 636 -> 628); one by one 2 % slower than left alone, pairs six ahead in between.
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
      }
      if (__any(!(sum <= kSumLimit))) {
        if (late) scale_late();   // P(it - 1) V(it - 1) is in
        move_maximum(largest(s_cur));
        scale_late();
        sum = weights(neg_mc);
        if (it - last_move < kMovesApart) watched = kWatched;
        last_move = it;
      }
      l_run[0] += sum;
      // K(it+2) replaces K(it), V(it) replaces V(it-2)
      if (has2) stash(kbuf + (it & 1) * KBYTES, KSTR, kreg);
      stash_v(vbuf + (it & 1) * VBYTES, vreg);
      __syncthreads();
    };

    const std::integral_constant<bool, true> steady;
    const std::integral_constant<bool, false> draining;
    if constexpr (STATE) blk0 = 0, blk1 = 1;
    for (int blk = blk0; blk < blk1; ++blk) {
      if (per_block || MIXED) Lk_b = ap->lk_blk[blk];
      kpos = PosDesc32{ap->kpos[blk].start0, ap->kpos[blk].len0, ap->kpos[blk].start1, ap->kpos[blk].len1};
      tr = visible_key_tiles<KT>(a.causal, a.qpos, kpos, Lk_b, tile_row0, tile_row1);
      na = tr.a1 - tr.a0;
      nt = na + (tr.b1 - tr.b0);
      if (!STATE && nt == 0) continue;   // nothing of this block is visible to the query tile (workgroup-uniform)
      {
        const UnmaskedTiles unmasked = unmasked_key_tiles(KT, a.causal, wave_live, MIXED, wave_qmin, kpos.start0, kpos.len0, kpos.start1,
                                                          kpos.len1, Lk_b, na, tr.b0, tr.b1);
        free_a = unmasked.a;
        free_b0 = unmasked.b0;
        free_b1 = unmasked.b1;
      }
      kg = (const char*)ap->k[blk] + kv_head_off;
      vg = (const char*)ap->v[blk] + (VT ? vt_head_off : kv_head_off);

      // ---- prologue: K(0), V(0), K(1) to LDS; scores of tile 0.  (Every step ends on a barrier, so the previous
      //      block's last reads of these buffers are over.)
      full_tiles = Lk_b / KT;
      full_extent = (KT - 1) * (int)row_bytes + HS * 2;
      ragged_extent = (Lk_b - full_tiles * KT - 1) * (int)row_bytes + HS * 2;   // (not used when there is no ragged tile)
      v_tile = tile_of(1);
      if constexpr (TRAILING) {
        if constexpr (STATE) load_state_sums();   // (K(0) and K(1) ahead of the accumulators, see below)
        if (nt > 0) {
          fetch(kg, tile_of(0), kreg);
          if (nt > 1) fetch(kg, v_tile, vreg);
        }
        if constexpr (STATE) load_state_acc();
        if (nt == 0) continue;
        stash(kbuf, KSTR, kreg);
        if (nt > 1) stash(kbuf + KBYTES, KSTR, vreg);
        __syncthreads();
        f32x16 s0[NQB][KB], s1[NQB][KB];   // scores of the current and of the next tile
        bf16x8 p0[PS], p1[PS];             // weights of the tile before and of the current one
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk) asm volatile("" : "=v"(s1[0][kbk]));   // (undefined, and says so: see below)
#pragma unroll
        for (int ks = 0; ks < PS; ++ks) asm volatile("" : "=v"(p0[ks]), "=v"(p1[ks]));
        qk(kbuf, s0);
        if constexpr (STATE) {
#pragma unroll
          for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(oacc[0][db]));
          settle(m_run[0]);
          settle(l_run[0]);
          neg_mc = (m_run[0] == -INFINITY) ? kNoMaximum : -m_run[0] * a.scale_log2;
        }
        __syncthreads();   // step 0 overwrites K buffer 0 with tile 2
        int it = 0;
        auto one = [&]() __attribute__((always_inline)) {
          trailing_step(draining, it, s0, s1, p0, p1);
#pragma unroll
          for (int ks = 0; ks < PS; ++ks) p0[ks] = p1[ks];
          if (it + 1 < nt) {
#pragma unroll
            for (int kbk = 0; kbk < KB; ++kbk) s0[0][kbk] = s1[0][kbk];
          }
          ++it;
        };
        one();
        for (; it + 3 < nt; it += 2) {
          trailing_step(steady, it, s0, s1, p0, p1);
          trailing_step(steady, it + 1, s1, s0, p1, p0);
        }
        while (it < nt) one();
        if (late) scale_late();   // P(nt - 2) V(nt - 2) is in
        last_move -= nt;   // (the next block's tiles are counted from 0 again)
        products_v(nt - 1, p0);   // (the next block's first V tile is stored two barriers from here)
        continue;
      }
      if constexpr (STATE) {
        // Loads return in their order: K(0) and K(1) go ahead of the state, 128 KiB per workgroup, 34 to 68 MiB that all
        // workgroups ask for at once and that took 11 us to arrive, and V(0), first wanted after the softmax, behind it.
        load_state_sums();
        if (nt > 0) {
          fetch(kg, tile_of(0), kreg);
          fetch(kg, nt > 1 ? v_tile : tile_of(0), vreg);
        }
        load_state_acc();
        if (nt == 0) continue;
        stash(kbuf, KSTR, kreg);
        stash(kbuf + KBYTES, KSTR, vreg);
        fetch_v(vg, tile_of(0), vreg);
      } else {
        fetch(kg, tile_of(0), kreg);
        fetch_v(vg, tile_of(0), vreg);
        stash(kbuf, KSTR, kreg);
        stash_v(vbuf, vreg);
        if (nt > 1) {
          fetch(kg, v_tile, kreg);
          stash(kbuf + KBYTES, KSTR, kreg);
        }
      }
      __syncthreads();
      f32x16 s0[NQB][KB], s1[NQB][KB];   // scores of the current and of the next tile
      // s1 starts undefined and says so: an empty asm "defines" it.  Otherwise the compiler carries its stale value
      // from the previous block and item around every loop (the draining steps below may leave it untouched), as a
      // zero-initialised 32-register tuple that it keeps in scratch.
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
        for (int kbk = 0; kbk < KB; ++kbk) asm volatile("" : "=v"(s1[qb][kbk]));
      qk(kbuf, s0);
      if constexpr (STATE) {   // the state has to have arrived before the loop (see settle), and V(0) be in LDS
#pragma unroll
        for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(oacc[0][db]));
        settle(m_run[0]);
        settle(l_run[0]);
        stash_v(vbuf, vreg);
      }
      __syncthreads();   // step 0 overwrites K buffer 0 with tile 2: every wave must have read tile 0 first

      int it = 0;
      for (; it + 3 < nt; it += 2) {   // two steps per trip so the score registers swap roles without copies
        step(steady, it, s0, s1);
        step(steady, it + 1, s1, s0);
      }
      for (; it < nt; ++it) {          // at most three tiles left
        step(draining, it, s0, s1);
        if (it + 1 < nt) {             // (the last step leaves s1 undefined: nothing may read it)
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
            for (int kbk = 0; kbk < KB; ++kbk) s0[qb][kbk] = s1[qb][kbk];
        }
      }
    }

    const ItemQueues queues = {ap->ticket_slot, n_items, (int)gridDim.x, ap->n_queues};
    unsigned own_ticket = kNoDraw;
    if (drawing && threadIdx.x == 0) own_ticket = queues.begin(empty_queues);
    // ---- epilogue: normalise, write O (a row that saw no key at all: l = 0 -> O = 0, LSE = -inf)
    // ---- write O (this lane: query l32, dims 32 db + 8 j + 4 hl + 0..3) and LSE
    static_assert(!LINES || TRAILING || NWAVES * kRowsLdsBytes <= 2 * (KBYTES + VBYTES), "the waves' rows fit where the tiles were");
    int end_tid = threadIdx.x;
    if constexpr (LINES) asm volatile("" : "+v"(end_tid));   // (what the rows' exchange derives from it is not kept across the tile loop either)
    const int end_lane = end_tid & 63;
    // (every step ends on a barrier: the tiles are no longer read; but the last P V of TRAILING comes behind it)
    char* const wave_lds = smem + (TRAILING ? 2 * (KBYTES + VBYTES) : 0) + __builtin_amdgcn_readfirstlane(end_tid >> 6) * kRowsLdsBytes;
    if (STATE && !ap->state_last) {
      // not the last ring step: the state goes back as it is (each store instruction of a wave fills 1 KiB)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 v4 = {oacc[0][db][4 * j], oacc[0][db][4 * j + 1], oacc[0][db][4 * j + 2], oacc[0][db][4 * j + 3]};
          *(f32x4*)(st_rec + ((db * 4 + j) * 64 + lane) * 4) = v4;
        }
      st_rec[DB * 16 * 64 + lane] = m_run[0];
      st_rec[DB * 16 * 64 + 64 + lane] = l_run[0];
    } else if (MIXED && per_block) {
      // a split item of a mixed launch: its partial result, fp32, dense
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        const float l_tot = both_halves_sum(l_run[qb]);
        const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
        const int qrow = wave_row0 + qb * 32 + l32;
        const int row0 = ap->part_row0[blk0], part_rows = a.Lq - row0;
        if (qrow < row_end && hl == 0)
          ap->lse_part[blk0][((size_t)b * a.hq + h) * part_rows + (qrow - row0)] = l_tot > 0.f ? m_run[qb] * a.scale + __logf(l_tot) : -INFINITY;
        const int base = wave_row0 + qb * 32;
        float* const dst = (float*)ap->o_part[blk0] + (((size_t)b * part_rows + (base - row0)) * a.hq + h) * HS;
        put_rows<float>(wave_lds, end_lane, oacc[qb], inv, [&](int, int col, const u32x4 (&v)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (const int r = 8 * i + (end_lane >> 3); base + r < row_end) *(u32x4*)(dst + (size_t)r * a.hq * HS + col) = v[i];
        });
      }
    } else
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const float l_tot = both_halves_sum(l_run[qb]);
      const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
      const int base = wave_row0 + qb * 32, qrow = base + l32;
      if constexpr (LINES) {
        // (where a row of O lies is worked out once, by the lane that has the row, and handed to those that store it)
        const long long at = (long long)qo_offset(a, b, min(qrow, row_end - 1), h, HS);
        long long row_at[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) row_at[i] = __shfl(at, 8 * i + (end_lane >> 3));
        put_rows<OutT>(wave_lds, end_lane, oacc[qb], inv, [&](int, int col, const u32x4 (&v)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (base + 8 * i + (end_lane >> 3) < row_end) *(u32x4_any*)((OutT*)a.o + row_at[i] + col) = v[i];
        });
      }
      if (qrow < row_end) {
        if constexpr (!LINES) {
          OutT* dst = per_block ? (OutT*)ap->o_part[blk0] + (((size_t)b * a.Lq + qrow) * a.hq + h) * HS + 4 * hl
                                : (OutT*)a.o + qo_offset(a, b, qrow, h, HS) + 4 * hl;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              f32x4 v4 = {oacc[qb][db][4 * j] * inv, oacc[qb][db][4 * j + 1] * inv, oacc[qb][db][4 * j + 2] * inv,
                          oacc[qb][db][4 * j + 3] * inv};
              OutT* d = dst + db * 32 + j * 8;
              if constexpr (sizeof(OutT) == 4) {
                *(f32x4*)d = v4;
              } else {
                u32x2 pk = {pack_bf16(v4[0], v4[1]), pack_bf16(v4[2], v4[3])};
                *(u32x2*)d = pk;
              }
            }
        }
        if (hl == 0) {
          const float lse = l_tot > 0.f ? m_run[qb] * a.scale + __logf(l_tot) : -INFINITY;
          ((per_block && !MIXED) ? ap->lse_part[blk0] : a.lse)[((size_t)b * a.hq + h) * a.Lq + qrow] = lse;
        }
      }
    }
    if (threadIdx.x == 0) {   // waits for the draw only: the stores were issued after it
      unsigned empty = empty_queues;
      next_item[turn] = drawing ? queues.finish(own_ticket, empty) : n_items;
      empty_queues = empty;
    }
  }   // next work item
}

// smallest and largest position of the rows [a, b) (pos_min and pos_max of attn_device.h, on the host)
inline int64_t host_pos_min(const PosDesc32& d, int64_t a, int64_t b) {
  int64_t m = INT64_MAX;
  if (a < d.len0) m = d.start0 + a;
  if (b > d.len0) m = std::min(m, d.start1 + std::max<int64_t>(a, d.len0) - d.len0);
  return m;
}
inline int64_t host_pos_max(const PosDesc32& d, int64_t a, int64_t b) {
  int64_t m = INT64_MIN;
  if (a < d.len0) m = d.start0 + std::min<int64_t>(b, d.len0) - 1;
  if (b > d.len0) m = std::max(m, d.start1 + b - 1 - d.len0);
  return m;
}

template <int HS, int NQB, int NWAVES, int KT, int WPE, typename OutT, bool STATE = false, bool VT = false, bool MIXED = false, bool TRAILING = false>
int launch_mfma(const AttnArgs& args, hipStream_t stream, const uint16_t* listed = nullptr, int n_listed = 0) {
  constexpr int BM = NWAVES * NQB * 32;
  constexpr int KSTR = HS * 2 + 48, VSTR = VT ? KT * 2 + 16 : HS * 2 + 64;
  constexpr size_t lds = 2 * ((size_t)KT * KSTR + (VT ? (size_t)HS * VSTR : (size_t)KT * VSTR)) + (MIXED && TRAILING ? NWAVES * kRowsLdsBytes : 0);
  static_assert(BM == 256, "RowTiles");
  std::conditional_t<STATE || MIXED, ListedArgs, AttnArgs> a;
  static_cast<AttnArgs&>(a) = args;
  if (STATE && a.n_blocks != 1) return USP_ERR_UNSUPPORTED;
  const RowTiles tiles(usp_posdesc{a.qpos.start0, a.qpos.len0, a.qpos.start1, a.qpos.len1}, a.Lq, a.causal && !STATE);
  a.n_qtiles = tiles.n;
  a.tiles_run0 = tiles.in_run0;
  int64_t grid = (int64_t)a.n_qtiles * a.hq * a.bs * (a.per_block ? a.n_blocks : 1);
  [[maybe_unused]] auto put = [&](int at, uint32_t entry) {
    if constexpr (STATE || MIXED) a.list[at / 2] = at % 2 ? a.list[at / 2] | entry << 16 : entry;
  };
  if constexpr (STATE || MIXED) a.n_listed = 0;
  if constexpr (STATE) {
    // A middle step of a step-by-step ring leaves the rows that see nothing of its block as they are (under the zigzag split
    // half of a rank's rows see nothing of most blocks): their tiles are no items.  Drawn and put back, they were 8 to 12 us
    // at the end of such a step of L = 32768, ring 8.
    if (a.causal && !a.state_first && !a.state_last && a.n_qtiles <= kMaxListedItems) {
      int n = 0;
      for (int t = a.n_qtiles - 1; t >= 0; --t) {   // heaviest first
        const int r0 = t * BM, r1 = std::min(a.Lq, r0 + BM);
        bool sees = false;
        for (int j = 0; j < a.n_blocks; ++j) sees = sees || host_pos_max(a.qpos, r0, r1) >= host_pos_min(a.kpos[j], 0, a.Lk);
        if (!sees) continue;
        put(n++, (uint32_t)t);
      }
      if (n == 0) return USP_OK;
      if (n < a.n_qtiles) {
        a.n_listed = n;
        grid = (int64_t)n * a.hq * a.bs;
      }
    }
  }
  if constexpr (MIXED) {
    if (a.n_split_tiles < 0 || a.n_split_tiles > a.n_qtiles) return USP_ERR_UNSUPPORTED;
    const int64_t split = (int64_t)a.n_split_tiles * a.hq * a.bs * a.n_blocks;
    grid = split + (int64_t)(a.n_qtiles - a.n_split_tiles) * a.hq * a.bs;
    if (split > 0x7fffffffll) return USP_ERR_UNSUPPORTED;
    a.n_split_items = (int)split;
    if (n_listed > 0) {
      if (n_listed > kMaxListedItems) return USP_ERR_UNSUPPORTED;
      for (int j = 0; j < n_listed; ++j) {
        const int tile = listed[j] & ((1 << kListedTileBits) - 1), piece = listed[j] >> kListedTileBits;
        if (tile >= a.n_qtiles) return USP_ERR_UNSUPPORTED;
        if (piece != kListedWhole && (piece >= a.n_blocks || tiles.begin(tile) < a.part_row0[piece])) return USP_ERR_UNSUPPORTED;
        put(j, listed[j]);
      }
      a.n_listed = n_listed;
      grid = (int64_t)n_listed * a.hq * a.bs;
    }
  }
  if (grid > 0x7fffffffll) return USP_ERR_UNSUPPORTED;
  auto kern = block_attn_fwd_mfma<HS, NQB, NWAVES, KT, WPE, OutT, STATE, VT, MIXED, TRAILING>;
  static LdsLimitRaised lds_limit;   // per kernel instance
  if (!raise_dynamic_lds_limit((const void*)kern, lds, lds_limit)) return USP_ERR_LAUNCH;
  // one workgroup per CU (its registers and LDS fill a CU), fewer when there are fewer items
  a.ticket_slot = ticket_slot_for(stream);
  a.n_items = (int)grid;
  a.n_queues = std::gcd(dev::kMaxItemQueues, a.bs * a.hkv);
  const int n_wgs = (int)std::min<int64_t>(grid, compute_units());
  hipLaunchKernelGGL(kern, dim3((unsigned)n_wgs), dim3(NWAVES * 64), lds, stream, a);
  return launch_status();
}

template <typename OutT, bool STATE = false, bool VT = false, bool MIXED = false>
int launch_mfma_64(const AttnArgs& a, hipStream_t stream, const uint16_t* listed = nullptr, int n_listed = 0) {
  const int64_t piece = std::accumulate(a.lk_blk, a.lk_blk + a.n_blocks, int64_t{0}) / a.n_blocks;
  return second_product_trails(a.Lk, piece) ? launch_mfma<64, 1, 8, 64, 2, OutT, STATE, VT, MIXED, true>(a, stream, listed, n_listed)
                                            : launch_mfma<64, 1, 8, 64, 2, OutT, STATE, VT, MIXED>(a, stream, listed, n_listed);
}

}  // namespace

int launch_ring_attn_fwd(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                         const usp_posdesc* kpos_blocks, int n_blocks, void* o, float* lse, int bs, int64_t Lq,
                         int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc& qpos,
                         int in_dtype, int o_dtype, hipStream_t stream, const SeqLayoutIO* seq, const RingState* state,
                         bool v_transposed) {
  if (n_blocks < 1 || n_blocks > kMaxBlocks) return USP_ERR_UNSUPPORTED;
  if (in_dtype != USP_BF16) return USP_ERR_DTYPE;
  AttnArgs a;
  a.seq_n = seq ? seq->rows_per_shard : 0;
  a.seq_heads = seq ? seq->heads : 0;
  a.seq_head0 = seq ? seq->head0 : 0;
  a.kv_pitch = seq && seq->kv_heads ? seq->kv_heads : hkv;
  a.q = q; a.o = o; a.lse = lse;
  for (int j = 0; j < kMaxBlocks; ++j) {
    const int jj = j < n_blocks ? j : 0;
    a.k[j] = k_blocks[jj];
    a.v[j] = v_blocks[jj];
    const usp_posdesc& kp = kpos_blocks[jj];
    a.kpos[j] = PosDesc32{(int)kp.start0, (int)kp.len0, (int)kp.start1, (int)kp.len1};
  }
  a.n_blocks = n_blocks;
  a.per_block = 0;
  a.n_split_items = a.n_split_tiles = 0;
  a.state = state ? state->state : nullptr;
  a.state_first = state ? state->first : 0;
  a.state_last = state ? state->last : 0;
  for (int j = 0; j < kMaxBlocks; ++j) {
    a.lk_blk[j] = (int)Lk;
    a.o_part[j] = nullptr;
    a.lse_part[j] = nullptr;
    a.part_row0[j] = 0;
  }
  a.bs = bs; a.hq = hq; a.hkv = hkv; a.g = hq / hkv;
  a.Lq = (int)Lq; a.Lk = (int)Lk;
  a.n_qtiles = a.tiles_run0 = 0;
  a.ticket_slot = 0;
  a.n_items = 0;
  a.n_queues = 1;
  a.causal = causal;
  a.scale = scale;
  a.scale_log2 = scale * 1.4426950408889634f;
  a.qpos = PosDesc32{(int)qpos.start0, (int)qpos.len0, (int)qpos.start1, (int)qpos.len1};
  if (state && v_transposed) return USP_ERR_UNSUPPORTED;
  if (v_transposed) {   // V blocks in key-tile-transposed layout (bf16 in and out)
    if (o_dtype != USP_BF16) return USP_ERR_DTYPE;
    return hs == 128 ? launch_mfma<128, 1, 8, 64, 2, __bf16, false, true>(a, stream)
                     : launch_mfma_64<__bf16, false, true>(a, stream);
  }
  if (a.state) {   // the instance that reads and writes the running state of a step-by-step ring
    if (hs == 128)
      return o_dtype == USP_FP32 ? launch_mfma<128, 1, 8, 64, 2, float, true>(a, stream)
                                 : launch_mfma<128, 1, 8, 64, 2, __bf16, true>(a, stream);
    return o_dtype == USP_FP32 ? launch_mfma_64<float, true>(a, stream)
                               : launch_mfma_64<__bf16, true>(a, stream);
  }
  // 256 query rows per workgroup (8 waves x 32), 64-key tiles, two waves per SIMD
  if (hs == 128)
    return o_dtype == USP_FP32 ? launch_mfma<128, 1, 8, 64, 2, float>(a, stream)
                               : launch_mfma<128, 1, 8, 64, 2, __bf16>(a, stream);
  if (o_dtype == USP_FP32) return launch_mfma_64<float>(a, stream);
  return launch_mfma_64<__bf16>(a, stream);
}

int launch_block_attn_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int bs, int64_t Lq,
                          int64_t Lk, int hq, int hkv, int hs, float scale, int causal, const usp_posdesc& qpos,
                          const usp_posdesc& kpos, int in_dtype, int o_dtype, hipStream_t stream, const RingState* state) {
  if (block_goes_to_waves(bs, Lq, Lk, hq, hs, causal, in_dtype))
    return launch_wave_split_block_fwd(q, k, v, o, lse, bs, Lq, Lk, hq, hkv, hs, scale, causal, qpos, kpos, in_dtype, o_dtype,
                                       stream, state);
  return launch_ring_attn_fwd(q, &k, &v, &kpos, 1, o, lse, bs, Lq, Lk, hq, hkv, hs, scale, causal, qpos, in_dtype,
                              o_dtype, stream, nullptr, state);
}

size_t attn_fwd_state_bytes(int bs, int64_t Lq, int hq, int hs) {
  // one record per 32-row block, query tiles of 256 rows rounded up (the kernel's item shape)
  return (size_t)bs * hq * (size_t)((Lq + 255) / 256) * 8 * state_record_floats(hs) * sizeof(float);
}

int launch_attn_fwd_partials(const void* q, const void* const* k_blocks, const void* const* v_blocks,
                             const usp_posdesc* kpos_blocks, const int* lk_blocks, int n_blocks, float* const* o_parts,
                             float* const* lse_parts, int bs, int64_t Lq, int64_t Lk, int hq, int hkv, int hs,
                             float scale, int causal, const usp_posdesc& qpos, hipStream_t stream,
                             const SeqLayoutIO* seq, const MixedLaunch* mixed) {
  if (n_blocks < 1 || n_blocks > kMaxBlocks) return USP_ERR_UNSUPPORTED;
  if (mixed && mixed->v_transposed)   // a piece of transposed tiles begins with a whole tile, 16-byte aligned
    for (int j = 0; j < n_blocks; ++j)
      if ((uintptr_t)v_blocks[j] & 15) return USP_ERR_UNSUPPORTED;
  AttnArgs a;
  a.seq_n = seq ? seq->rows_per_shard : 0;
  a.seq_heads = seq ? seq->heads : 0;
  a.seq_head0 = seq ? seq->head0 : 0;
  a.kv_pitch = seq && seq->kv_heads ? seq->kv_heads : hkv;
  a.q = q; a.o = nullptr; a.lse = nullptr;
  for (int j = 0; j < kMaxBlocks; ++j) {
    const int jj = j < n_blocks ? j : 0;
    a.k[j] = k_blocks[jj];
    a.v[j] = v_blocks[jj];
    const usp_posdesc& kp = kpos_blocks[jj];
    a.kpos[j] = PosDesc32{(int)kp.start0, (int)kp.len0, (int)kp.start1, (int)kp.len1};
    a.lk_blk[j] = lk_blocks ? lk_blocks[jj] : (int)Lk;
    if (a.lk_blk[j] < 1 || a.lk_blk[j] > Lk) return USP_ERR_SHAPE;
    a.o_part[j] = o_parts[jj];
    a.lse_part[j] = lse_parts[jj];
    a.part_row0[j] = mixed && mixed->part_row0 ? (int)mixed->part_row0[jj] : 0;
    if (a.part_row0[j] < 0 || a.part_row0[j] > Lq) return USP_ERR_SHAPE;
  }
  a.n_blocks = n_blocks;
  a.per_block = 1;
  a.n_split_items = a.n_split_tiles = 0;
  a.state = nullptr;
  a.state_first = a.state_last = 0;
  a.bs = bs; a.hq = hq; a.hkv = hkv; a.g = hq / hkv;
  a.Lq = (int)Lq; a.Lk = (int)Lk;
  a.n_qtiles = a.tiles_run0 = 0;
  a.ticket_slot = 0;
  a.n_items = 0;
  a.n_queues = 1;
  a.causal = causal;
  a.scale = scale;
  a.scale_log2 = scale * 1.4426950408889634f;
  a.qpos = PosDesc32{(int)qpos.start0, (int)qpos.len0, (int)qpos.start1, (int)qpos.len1};
  if (mixed) {
    a.o = mixed->o;
    a.lse = mixed->lse;
    a.per_block = 0;
    a.n_split_tiles = mixed->n_split_tiles;
    auto go = [&](auto launch) { return launch(a, stream, mixed->listed, mixed->n_listed); };
    if (mixed->v_transposed)
      return hs == 128 ? go(launch_mfma<128, 1, 8, 64, 2, __bf16, false, true, true>)
                       : go(launch_mfma_64<__bf16, false, true, true>);
    return hs == 128 ? go(launch_mfma<128, 1, 8, 64, 2, __bf16, false, false, true>)
                     : go(launch_mfma_64<__bf16, false, false, true>);
  }
  return hs == 128 ? launch_mfma<128, 1, 8, 64, 2, float>(a, stream) : launch_mfma_64<float>(a, stream);
}

}  // namespace usp
