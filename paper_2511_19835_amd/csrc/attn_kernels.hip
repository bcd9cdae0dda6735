// Block-sparse flash attention with the rectification fused into the epilogue
// (paper Sec. 3.1 sparse attention, Alg. 1 steps 16-17; Sec. 4.1 / 4.2, Alg. 1 steps 19-23).
//
// The kernel is persistent: one workgroup of eight waves per CU, in groups of BLK/32 waves (two groups
// at BLK = 128, four at BLK = 64; one wave per 32 query rows; groups g and g + NGRP/2 on the same
// SIMDs). A group works through a sequence of items -- query blocks of some (batch, head) -- that
// schedule_kernel dealt to it, as one unbroken stream of steps: a video query block walks its
// compact, ascending list of critical key blocks, a text query block (and every block under
// RSA_DENSE) all M key blocks, KVS keys per step. For each step the K rows [KVS][d] and the
// channel-major V rows [d][KVS] (HALVES, see attn_kernel: half of the channels of all keys of the block,
// [d/2][BLK]) are brought into the group's own LDS rings by direct-to-LDS loads
// (global_load_lds_dwordx4: no staging registers), one step ahead -- also across the boundary
// between two items, so the matrix pipe never drains. Each wave computes, with
// v_mfma_f32_16x16x32_bf16,
//     S^T = K Q^T      (M = key, N = query, k = channel)      -> accumulators: two query columns per lane,
//     O^T += V^T P^T   (M = channel, N = query, k = key)         one of either query tile of 16
// so the online softmax is lane-local except for sums over four lanes at the end of an item,
// and the probabilities a lane holds after the first product are exactly the B operand it
// needs for the second (rsa_pool stores V in that key order, and the K operands take their rows
// to match, key_row).
//
// What bounds it is the power that the chip may draw, and the instruction decides what a product costs of it. In a loop of
// the same two phases without loads of tiles, 16 x 16 x 32 sustains 1600 TFLOP/s and 32 x 32 x 16 1470 (2308 and 2206
// cycles a step at 1.72 and 1.50 GHz; products alone from registers 2050 and 1785). The price is the vector ALU's: beside
// products of 16 x 16 it issues two instructions in 16 cycles, so that the softmax phase is now the longer of the two,
// and requests are all made in the MFMA phase. Against the larger instruction, us, the attention entry point, both forms in turn
// (two figures: two boxes): 24 heads of 931 blocks, lists of 94, 14 790, 14 710 and 14 360, 14 080; 3 heads 1904 and 1783; 40 of 591
// 9865 and 9469; 24 of 159, lists of 16, 479 and 452, all blocks 4099 and 3747; d = 64, 2 x 12 of 160, lists of 40, 715 and 675;
// blocks of 64, 24 of 1182 7065 and 6878, all of 380 6282 and 5861. Where power is not the bound the larger one is the
// faster: half a round of blocks of 64 (1 head of 512, lists of 52) 102.3 and 106.6; where the fabric is (24 of 931, full mask
// rule) a loop of launches takes 21 060, 20 700, 20 870 and 21 450, 21 200, 20 900, four launches on their own 21 600 and 20 900.
//
// A step of a group is two phases, separated by workgroup barriers: an MFMA phase (the P V
// product of the previous step, then K Q^T of this one: matrix instructions, their LDS operand
// reads a few slots ahead and the requests for the next tile, between the two products of a slot) and a softmax phase
// (VALU only). The groups run one barrier apart, so that on every SIMD one wave feeds the matrix
// pipe while the other uses the VALU. When an item ends its output is written in the softmax phase
// of the next item's first step (HALVES: its second): O = R_n * acc / l + C_n, C_n = sum_{m: not kept and M_c}
// A^pool[n][m] v^pool_m (computed beforehand by compensation_kernel into the workspace).
//
// 4*B*B*d flop per (query block, key block) pair against 2*B*d*2 bytes of K/V traffic.
// The small kernels around this one are in attn_side_kernels.hip. row_rank_kernel orders the video query
// blocks of a head by their first three kept key blocks; schedule_kernel deals that order to the groups so
// that each XCD (workgroup id modulo 8) owns contiguous ranges of it, of a whole head at a time where the
// caches hold the heads at work, and groups resident together walk similar lists and share K/V tiles in the
// XCD's L2. With few rounds of items the rows of the last round and the text rows are cut into pieces, where
// that is faster, and all groups end at about the same key block (merge_kernel adds the pieces); with many,
// the text rows go first and the groups end within one item of each other.
#include "attn_sched.hpp"
#include "lds_dma.hpp"
#include "rsa_common.hpp"

namespace rsa {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr int KSTAGES = 2;          // LDS ring depth of the K tiles of a group (the loop is unrolled over it)
constexpr int VSTAGES = 3;          // ... of its V^T tiles, which are read one phase later than the K tile of the same step
#ifndef RSA_MWIN
#define RSA_MWIN 4
#endif
constexpr int MWIN = RSA_MWIN;      // MFMA slots between the LDS read of a K operand and its use

template <int D, int BLK, bool HALVES>
struct AttnCfg {
  static constexpr int NW = BLK / 32;       // waves per group (one per 32 query rows)
  static constexpr int NGRP = 8 / NW;       // groups = query blocks per workgroup: eight waves, two per SIMD
  static constexpr int NTHR = 64 * NW * NGRP;
  // keys per step: half a key block, so that every key block is two steps and every item an even
  // number of them (the loop over the steps is unrolled twice)
  static constexpr int KVS = BLK / 2;
  static constexpr int SPB = BLK / KVS;     // steps per key block
  static constexpr int KT = KVS / 16;       // key tiles of S^T per step
  static constexpr int KS = D / 32;         // k-steps of K Q^T
  static constexpr int DT = D / 16;         // channel tiles of O^T
  static constexpr int PC = KVS / 32;       // 32-key chunks per step
  static constexpr bool VH = HALVES;        // V^T by halves of the channels, all keys of the block at once (see attn_kernel)
  static constexpr int PPC = VH ? BLK / 32 : PC;     // 32-key chunks of one P V product
  static constexpr int PDT = VH ? DT / 2 : DT;       // ... and its channel tiles
  static constexpr int KCPR = D / 8;        // 16-byte chunks per K row
  static constexpr int VCPR = PPC * 4;      // 16-byte chunks per V^T row of a tile
  static constexpr int VROWS = PDT * 16;    // V^T rows of a tile
  static constexpr int KINST = KVS * KCPR / 64;   // 1 KB direct-to-LDS loads per K step tile
  static constexpr int VINST = VROWS * VCPR / 64; // ... per V^T step tile
  static constexpr int KPW = KINST / NW;    // per wave
  static constexpr int VPW = VINST / NW;
  static constexpr int KBUF = KVS * KCPR;   // 16-byte chunks per K buffer
  static constexpr int VBUF = VROWS * VCPR; // ... per V^T buffer
  static constexpr int GROUP = KSTAGES * KBUF + VSTAGES * VBUF;   // 16-byte chunks of one group: [K stages | V^T stages]
  static_assert(!VH || SPB * PDT == DT, "a half of the channels for each step of a block");
  static_assert(KINST % NW == 0 && VINST % NW == 0, "loads must split evenly over the waves");
  static_assert(NGRP * GROUP * 16 <= 160 * 1024, "the rings of all groups must fit the LDS of a CU");
  static_assert(SPB == 2, "the main loop is unrolled twice: over the K stages and over the steps of a key block");
  static_assert(NGRP % 2 == 0 && BLK % KVS == 0, "groups pair up on the SIMDs; a block is a whole number of steps");
};

// LDS tiles are unpadded; the 16-byte chunk c of row r is stored at chunk position c ^ key(r) so that the 16 rows of an
// operand, read at one logical chunk index, hit 16 different positions (all banks once), and also where an access takes
// four rows each from lanes whose chunk indices differ in their lowest bit. CPR = chunks per row (4, 8 or 16). V^T operands
// are 16 consecutive rows, K operands the rows key_row below: eight consecutive ones and the eight that are 16 further on.
template <int CPR>
__device__ __forceinline__ int swz_v_key(int r) {
  if constexpr (CPR == 4) return ((r / 4 ^ r / 8) & 1) * 2 | (r / 8 & 1);
  return (r / (16 / CPR)) & (CPR - 1);
}
template <int CPR>
__device__ __forceinline__ int swz_k_key(int r) { return CPR == 16 ? (r & 7) | (r & 16) / 2 : (r / 2 & 3) | (r & 16) / 4; }
// Row of a run of 32 keys that lane row i of a K operand takes (its partner operand: 8 further on): the keys whose scores
// a lane then holds, four from either operand, are the eight of its B operand in the order that rsa_pool stores V^T in.
__device__ __forceinline__ int key_row(int i) { return (i & 7) + 2 * (i & 8); }

// Values that the four lanes of a query column (lane l, l ^ 16, l ^ 32, l ^ 48) hold, put together with
// v_permlane16_swap and v_permlane32_swap; all four get the same bits.
// The vector elements are copied to scalars before the bit casts: a bit cast applied
// directly to an element expression reads element 0 whatever the index.
template <class F>
__device__ __forceinline__ float over_column(float v, F&& f) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t a0 = a[0], a1 = a[1];
  const uint32_t w = __builtin_bit_cast(uint32_t, f(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1)));
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  const uint32_t b0 = b[0], b1 = b[1];
  return f(__builtin_bit_cast(float, b0), __builtin_bit_cast(float, b1));
}
__device__ __forceinline__ float column_max(float v) {
  return over_column(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float column_sum(float v) {
  return over_column(v, [](float a, float b) { return a + b; });
}

// Matrix products as inline asm, because only there the accumulator can be held to its place: the compiler gives this
// instruction a destination of its own, and the accumulators then wander through the registers and into scratch. Its hazards
// are ours in return: an accumulator is used by the next product at the earliest four products on (the matrix pipe needs 16
// cycles, four wait states, for each), and before any other use stands settle_products. Operands come from LDS reads (waited
// for) and from the phase before (a barrier away). tests/test_product_waits.py holds the compiler's output to all three.
__device__ __forceinline__ void mfma_add(floatx4& c, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_first(floatx4& c, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
}
// The products into c[][] are complete (a result of four passes may be touched by another instruction eight wait states on:
// NOPS, and four for each product that followed).
template <int NOPS, int N>
__device__ __forceinline__ void settle_products(floatx4 (&c)[N][2]) {
  asm volatile("s_nop %0" ::"n"(NOPS - 1) : "memory");
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(c[i][0]), "+v"(c[i][1]));
}

// The lane number, worked out where it is asked for. What happens once per item (query rows, epilogue)
// takes its lane-dependent addresses from this: values derived from the lane number at the top of the
// kernel would be live across the whole step loop, where there is no register left for them, and a
// spilled vector register comes back with a wait for every load in flight, tile requests included.
__device__ __forceinline__ int lane_now() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// The running softmax reference only moves when a score is more than this many binades away from it
// (above it; in the first step of an item, either way): probabilities then stay within 2^+-kLazyBits of
// one another's scale, far inside what fp32 sums and bf16 operands hold, and the accumulators are
// rescaled very rarely.
constexpr float kLazyBits = 40.0f;

template <int V>
struct IntC { static constexpr int value = V; };
// f(IntC<I>{}) for I = FROM .. TO-1, unrolled at compile time (the index is a constant inside f)
template <int FROM, int TO, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (FROM < TO) {
    f(IntC<FROM>{});
    static_for<FROM + 1, TO>(f);
  }
}

// Work of the persistent attention kernel. An item is one query block of one (batch, head); a slot
// is one group of waves of one resident workgroup and works through a sequence of items.
//   table != NULL: schedule_kernel dealt the items to the slots (balanced by their number of steps,
//                  neighbouring rows of the launch order to neighbouring slots at the same time; an item may be
//                  part of a row, whose result goes to a piece buffer for merge_kernel);
//   table == NULL: item i goes to slot i % n_slots (no workspace: index order).
struct SchedArgs {
  const int2* table;        // [slots][cap] entries (attn_sched.hpp)
  const int32_t* nitems;    // [slots]
  const int32_t* total;     // [slots] key blocks of all items of the slot
  const int32_t* piece0;    // [slots] the slot's first piece buffer within its queue
  float* pieces;
  int cap, slots_per_queue, pieces_per_queue;
  int n_items, n_dense;     // all items; the dense ones (text query blocks, or every block under RSA_DENSE) come first
  int dense_per_bh, dense_first;
};

// HALVES (blocks of 64): a V^T row of a key block is 128 bytes, one line, and the 32 keys of a step are half of it. Taken
// step by step every line is asked for twice, and a step in the sparse layers waited 430 cycles for its tiles (24 heads of
// 1182 blocks at d = 128: 1.23e9 requests of the L2, 55 GB through the fabric at 6 TB/s). So the two P V products of a
// block take all its 64 keys and half of the channels each, one step later: M(s) multiplies the probabilities of the
// block before with the half s % 2 of its V^T rows, whole lines. Probabilities of the block's first step are kept aside (pbn)
// while the second product of the block before still needs pb, and an item's output is complete, and written, in the second
// step of the next. Attention of that layer 8150 -> 6780 us, 24 heads of 317 blocks 559 -> 538. Not for RSA_DENSE, where
// the groups of a CU walk in step and the L1 serves the second half (317 blocks: 4313 -> 4457), nor at d = 64, where the
// softmax hides the requests and the moves do not (24 heads of 1182: 4297 -> 4458). The bits of the output are those of the
// step-by-step form as long as the softmax reference stays at 0; where it moves, it is rounded up to a whole number here,
// so that probabilities that wait can follow it in their exponents (below 2^-126 they become 0).
template <int D, int BLK, bool HALVES>
__global__ __launch_bounds__(512, 1) void attn_kernel(Dims dm, AttnArgs a, SchedArgs sc) {
  using C = AttnCfg<D, BLK, HALVES>;
  constexpr int KBUF = C::KBUF;
  constexpr int KVS = C::KVS, NGRP = C::NGRP;
  __shared__ u32x4 lds_all[NGRP * C::GROUP];   // per group: KSTAGES K tiles [KVS][d], then VSTAGES V^T tiles [d][KVS]

  const bool dense_all = (a.flags & RSA_DENSE) != 0;
  const int tid = threadIdx.x;
  const int wave_wg = __builtin_amdgcn_readfirstlane(tid / 64);
  const int grp = wave_wg / C::NW;                   // which group of this workgroup
  const int wave = wave_wg % C::NW;                  // wave inside the group (groups g and g + NGRP/2 share their SIMDs)
  const int lane = tid % 64;
  const int l16 = lane % 16, g4 = lane / 16;         // query column (of either query tile) and k-group of this lane
  u32x4* lds = lds_all + grp * C::GROUP;

  // ---- the items of this group, and how many rounds the workgroup turns -------------------
  // Slots are numbered so that the slots of one schedule queue sit on one XCD (workgroup id
  // modulo 8) and the groups of a workgroup are neighbours in it.
  const int n_wg = gridDim.x, wg = blockIdx.x;
  auto slot_of_group = [&](int g) __attribute__((always_inline)) {
    if (!sc.table) return wg * NGRP + g;
    return (wg % 8) * sc.slots_per_queue + (wg / 8) * NGRP + g;
  };
  const int n_slots = n_wg * NGRP;                   // (index-order dealing)
  auto record_of_item = [&](int i) __attribute__((always_inline)) {       // index order: dense items, then video rows
    int bhx, qbx;
    if (i < sc.n_dense) {
      bhx = i / sc.dense_per_bh;
      qbx = sc.dense_first + i % sc.dense_per_bh;
    } else {
      const int v = i - sc.n_dense;
      bhx = v / dm.n;
      qbx = v % dm.n;
    }
    return bhx * RSA_MAX_BLOCKS + qbx;
  };
  auto blocks_of_record = [&](int rec) __attribute__((always_inline)) {
    const int bhx = rec / RSA_MAX_BLOCKS, qbx = rec % RSA_MAX_BLOCKS;
    const bool sp = !dense_all && qbx < dm.n;
    return sp ? list_length(a, dm, (size_t)bhx * dm.n + qbx) : dm.m;
  };
  const int slot = slot_of_group(grp);
  int n_my_items, wg_rounds = 0;
  if (sc.table) {
    n_my_items = sc.nitems[slot];
#pragma unroll
    for (int g = 0; g < NGRP; ++g) {
      const int t = sc.total[slot_of_group(g)];
      wg_rounds = max(wg_rounds, t > 0 ? t * C::SPB + 1 : 0);
    }
  } else {
    n_my_items = slot < sc.n_items ? (sc.n_items - slot + n_slots - 1) / n_slots : 0;
#pragma unroll
    for (int g = 0; g < NGRP; ++g) {
      int t = 0;
      for (int i = wg * NGRP + g; i < sc.n_items; i += n_slots) t += blocks_of_record(record_of_item(i));
      wg_rounds = max(wg_rounds, t > 0 ? t * C::SPB + 1 : 0);
    }
  }
  if (wg_rounds == 0) return;                        // the whole workgroup: nothing was dealt to it
  // k-th entry of this group: record and span. Scalar loads (one with a table), so that it can be asked for
  // well ahead of make_item.
  struct Entry { int rec, span; };
  auto my_entry = [&](int k) __attribute__((always_inline)) {
    typedef const int32_t __attribute__((address_space(4))) * const_i32_t;
    Entry e;
    if (sc.table) {
      const const_i32_t p = (const_i32_t)(uintptr_t)sc.table + ((size_t)slot * sc.cap + k) * 2;
      e.rec = p[0];
      e.span = p[1];
    } else {
      e.rec = record_of_item(slot + k * n_slots);
      e.span = make_span(0, blocks_of_record(e.rec), false);
    }
    return e;
  };

  // What the phases need to know of an item: all wave-uniform.
  typedef const int32_t __attribute__((address_space(4))) * const_list_t;
  struct Item {
    int bh, qb;
    int ns;                 // steps: SPB per entry of its span
    int span;               // its span of the list (a dense row: of the M key blocks)
    int has_list;
    const_list_t list;      // the entries of its span; a dense row: any readable address
    uint64_t Kbytes, Vtbytes;   // K rows and V^T tiles of its (batch, head)
    int64_t qo_off;         // element offset of its first query row in Q and in O
    int q_t0, q_count;      // its first token and how many it has
  };
  auto make_item = [&](const Entry& en) __attribute__((always_inline)) {
    Item it;
    it.bh = en.rec / RSA_MAX_BLOCKS;
    it.qb = en.rec % RSA_MAX_BLOCKS;
    const bool sp = !dense_all && it.qb < dm.n;
    const size_t vrow = (size_t)it.bh * dm.n + it.qb;
    it.span = en.span;
    it.ns = span_len(en.span) * C::SPB;
    it.has_list = sp ? 1 : 0;
    const int b = it.bh / dm.heads, h = it.bh % dm.heads;
    const int64_t base = (int64_t)b * dm.sb + (int64_t)h * dm.sh;
    // (with RSA_DENSE every list pointer may be NULL: a dense row reads the first word of Q instead)
    it.list = (const_list_t)(uintptr_t)(sp ? (const void*)(a.block_idx + vrow * dm.m + span_first(en.span)) : (const void*)a.Q);
    it.Kbytes = (uint64_t)(uintptr_t)(a.K + base);
    it.Vtbytes = (uint64_t)(uintptr_t)(a.Vt + (size_t)it.bh * dm.m * D * BLK);
    const int64_t t0 = dm.block_start(it.qb);
    it.q_t0 = (int)t0;
    it.q_count = dm.block_count(it.qb);
    it.qo_off = base + t0 * dm.st;
    return it;
  };
  auto load_item = [&](int k) __attribute__((always_inline)) { return make_item(my_entry(k)); };

  // ---- direct-to-LDS loads ---------------------------------------------------------------
  // A load fills 1 KB of LDS = RK consecutive K rows (RV consecutive V^T rows). Load ii of
  // wave w covers rows pass*ROWS_PER_PASS + (class*NW + w)*RK + (lane / chunks-per-row): the
  // swizzle key of a lane's row then depends on the class only (it repeats every 32 K rows and every 16 V^T
  // rows), so KOFF (VOFF: 1) per-lane byte offsets serve all of a wave's loads and everything else is scalar.
  constexpr int RK = 64 / C::KCPR, RV = 64 / C::VCPR;
  constexpr int KOFF = (C::NW * RK >= 32) ? 1 : 32 / (C::NW * RK);
  constexpr int VOFF = (C::NW * RV >= 16) ? 1 : 16 / (C::NW * RV);
  static_assert(C::KPW % KOFF == 0 && C::VPW % VOFF == 0, "row classes must divide a wave's loads");
  int k_r0[KOFF], k_col[KOFF];
  uint32_t k_voff[KOFF], v_voff[VOFF];
#pragma unroll
  for (int c = 0; c < KOFF; ++c) {
    k_r0[c] = (c * C::NW + wave) * RK + lane / C::KCPR;
    k_col[c] = ((lane % C::KCPR) ^ swz_k_key<C::KCPR>(k_r0[c])) * 8;              // element offset in the row
    k_voff[c] = (uint32_t)((k_r0[c] * dm.st + k_col[c]) * 2);
  }
#pragma unroll
  for (int c = 0; c < VOFF; ++c) {
    const int r0 = (c * C::NW + wave) * RV + lane / C::VCPR;
    v_voff[c] = (uint32_t)((r0 * BLK + ((lane % C::VCPR) ^ swz_v_key<C::VCPR>(r0)) * 8) * 2);
  }
  constexpr int K_ROWS_PER_PASS = C::NW * RK * KOFF, V_ROWS_PER_PASS = C::NW * RV * VOFF;
  constexpr int K_LDS_CLASS = C::NW * RK * C::KCPR * 16, V_LDS_CLASS = C::NW * RV * C::VCPR * 16;
  constexpr int K_LDS_PASS = K_ROWS_PER_PASS * C::KCPR * 16, V_LDS_PASS = V_ROWS_PER_PASS * C::VCPR * 16;
  const uint32_t ldsK_addr = (uint32_t)(uintptr_t)lds + wave * RK * (C::KCPR * 16);
  const uint32_t ldsV_addr = (uint32_t)(uintptr_t)lds + KSTAGES * KBUF * 16 + wave * RV * (C::VCPR * 16);

  // Requests for the K rows and the V^T rows of one step. Everything that does not depend on the
  // step is worked out once, in bytes: load ii of a wave is a per-lane byte offset (kvo / vvo, the
  // pass folded in) from the tile's scalar base and a constant LDS offset from the stage's scalar
  // base, so that a request is one scalar add into M0 and the load itself, and a tile is prepared
  // from its block index with a dozen scalar instructions.
  const uint32_t kblock_bytes = (uint32_t)BLK * (uint32_t)dm.st * 2u;       // K rows of consecutive key blocks
  const uint32_t kstep_bytes = (uint32_t)KVS * (uint32_t)dm.st * 2u;        // ... of consecutive steps inside a block
  const uint32_t kpass_bytes = (uint32_t)K_ROWS_PER_PASS * (uint32_t)dm.st * 2u;
  const int64_t text_adjust = ((int64_t)dm.tv - (int64_t)dm.n * BLK) * dm.st * 2;   // text blocks start at T_v, not N*B
  const int last_video_count = dm.block_count(dm.n - 1), last_count = dm.block_count(dm.m - 1);
  constexpr uint32_t kVtBlockBytes = (uint32_t)D * BLK * 2u;
  constexpr int LPS = C::KPW + C::VPW;           // loads per step per wave
  uint32_t kvo[C::KPW], vvo[C::VPW];             // per-lane byte offsets of this wave's loads of a full tile
#pragma unroll
  for (int ii = 0; ii < C::KPW; ++ii) kvo[ii] = k_voff[ii % KOFF] + (uint32_t)(ii / KOFF) * kpass_bytes;
#pragma unroll
  for (int ii = 0; ii < C::VPW; ++ii) vvo[ii] = v_voff[ii % VOFF] + (uint32_t)((ii / VOFF) * (V_ROWS_PER_PASS * BLK * 2));
  struct Tile {
    uint64_t kp;          // K rows of this step
    uint64_t vp;          // V^T rows of this step
    uint32_t kdst, vdst;  // LDS byte addresses of this wave's first load into the stage
    uint32_t klast;       // byte offset of the block's last row from kp
    uint32_t koff[C::KPW];   // kvo, held to the rows of the block
  };
  // The key block whose tiles are being requested: start of its K rows and V^T rows, valid keys.
  uint64_t blk_kp = 0, blk_vp = 0;
  int blk_count = BLK;
  const uint32_t krow_bytes = (uint32_t)dm.st * 2u;
  // A tile is prepared in pieces of two or three instructions each, so that the caller can put one between the two MFMAs of
  // each of its slots: a matrix instruction covers 16 cycles and a wave issues an instruction every five or so, so that with
  // all forty in one place (or four behind every second MFMA) the matrix pipe stood still. Pieces 0 .. kOpenPieces-1 open the
  // key block m (first step of a block), the step pieces after them are taken for every step.
  // In a ragged key block (the last video block, the last text block) rows past its end re-read its last row (masked
  // later; V^T is zero-padded in HBM): the byte offset of every lane is held to that row's, without a branch.
  constexpr int kOpenPieces = 7, kStepPieces = 6 + KOFF;
  uint64_t open_base = 0, open_off = 0;
  int open_count = BLK;
  auto open_piece = [&](auto pc, int m, uint64_t Kbytes, uint64_t Vtbytes) __attribute__((always_inline)) {
    constexpr int piece = decltype(pc)::value;
    if constexpr (piece == 0) open_off = (uint64_t)(m >= dm.n ? text_adjust : 0);
    if constexpr (piece == 1) open_base = Kbytes + open_off;
    if constexpr (piece == 2) open_off = (uint64_t)(uint32_t)m * kblock_bytes;
    if constexpr (piece == 3) blk_kp = open_base + open_off;
    if constexpr (piece == 4) open_count = m == dm.n - 1 ? last_video_count : BLK;
    if constexpr (piece == 5) blk_count = m == dm.m - 1 ? last_count : open_count;
    if constexpr (piece == 6) blk_vp = Vtbytes + (uint64_t)(uint32_t)m * kVtBlockBytes;
  };
  uint32_t step_skip = 0;
  auto step_piece = [&](auto pc, Tile& t, auto partc, int kst, int vst) __attribute__((always_inline)) {
    constexpr int piece = decltype(pc)::value;
    constexpr int part = decltype(partc)::value;
    // (a block that ends before its second step: the step reads the rows of the first, all of them masked)
    if constexpr (piece == 0) step_skip = part > 0 && blk_count > part * KVS ? part * kstep_bytes : 0u;
    if constexpr (piece == 1) t.kp = blk_kp + step_skip;
    if constexpr (piece == 2) t.klast = (uint32_t)(blk_count - 1) * krow_bytes - step_skip;
    if constexpr (piece == 3) t.kdst = ldsK_addr + kst * (KBUF * 16);
    if constexpr (piece >= 4 && piece < 4 + KOFF) {
      constexpr int c = piece - 4;
      const uint32_t last = t.klast + (uint32_t)k_col[c] * 2u;
#pragma unroll
      for (int ii = c; ii < C::KPW; ii += KOFF) t.koff[ii] = min(kvo[ii], last);
    }
    if constexpr (piece == 4 + KOFF) t.vp = blk_vp + part * (C::VH ? C::VROWS * BLK * 2u : KVS * 2u);
    if constexpr (piece == 5 + KOFF) t.vdst = ldsV_addr + vst * (C::VBUF * 16);
  };
  auto issue_load = [&](const Tile& t, auto idxc) __attribute__((always_inline)) {
    constexpr int idx = decltype(idxc)::value;
    if constexpr (idx < C::KPW) {
      constexpr int ii = idx;
      dma16_sv_imm<(ii / KOFF) * K_LDS_PASS + (ii % KOFF) * K_LDS_CLASS>(t.kdst, t.kp, t.koff[ii], lds);
    } else {
      constexpr int ii = idx - C::KPW;
      dma16_sv_imm<(ii / VOFF) * V_LDS_PASS + (ii % VOFF) * V_LDS_CLASS>(t.vdst, t.vp, vvo[ii], lds);
    }
  };

  // ---- loop-invariant LDS read positions (16-byte chunk index inside stage 0, tile 0) ----
  const u32x4* kread[C::KS];
  const u32x4* vread[C::PPC];
#pragma unroll
  for (int ks = 0; ks < C::KS; ++ks)
    kread[ks] = lds + key_row(l16) * C::KCPR + ((4 * ks + g4) ^ swz_k_key<C::KCPR>(key_row(l16)));
#pragma unroll
  for (int pc = 0; pc < C::PPC; ++pc)
    vread[pc] = lds + KSTAGES * KBUF + l16 * C::VCPR + ((4 * pc + g4) ^ swz_v_key<C::VCPR>(l16));

  // ---- the item being computed, the one after it, and the one whose output is still to be written
  Item cur = {}, nxt = {};
  int nxt_valid = 0, k_next = 0;       // k_next: the first item not yet loaded
  Entry ahead = {};                    // ... and its entry, read an item ahead
  // what the epilogue needs of the item that has just ended
  int done_bh = 0, done_sparse = 0, done_q_t0 = 0, done_q_count = 0;
  int done_piece = -1;                                       // piece buffer it goes to (-1: to O),
  int next_piece = sc.table ? sc.piece0[slot] : 0;           // and the next one free
  int64_t done_qo_off = 0;

  // Q as the B operand of S^T = K Q^T, resident in registers; the next item's rows come into registers of their own, a
  // step ahead: they come from HBM, and asked for behind the last K Q^T, with nothing but a softmax before their use, they kept
  // both groups waiting for some 5000 cycles of every item (with products of 32 x 32 x 16: 24 heads of 931 blocks, lists of 94, 14642 us
  // and 14532; 591 blocks, lists of 60: 9828 and 9755; shorter lists 0.2 %; where the power limit or the fabric bounds the kernel,
  // equal). Rows past
  // the end of a ragged block repeat its last row: the number of loads in flight is the same for every wave, and the waits
  // below count on it.
  bf16x8 qreg[C::KS][2], qnext[C::KS][2];      // (k-step, query tile)
  const float cs = dm.scale * kLog2e;   // scores -> binades
  auto load_q = [&](bf16x8 (&dst)[C::KS][2], int64_t qo_off, int q_count) __attribute__((always_inline)) {
    const int ln = lane_now();
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const int q = min(wave * 32 + 16 * f + ln % 16, q_count - 1);
      const uint16_t* qrow = a.Q + qo_off + (int64_t)q * dm.st + 8 * (ln / 16);
#pragma unroll
      for (int s = 0; s < C::KS; ++s) dst[s][f] = *reinterpret_cast<const bf16x8*>(qrow + 32 * s);
    }
  };
#pragma unroll
  for (int s = 0; s < C::KS; ++s)
#pragma unroll
    for (int f = 0; f < 2; ++f) qnext[s][f] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
  const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
  floatx4 oacc[C::DT][2];                // (channel tile, query tile)
#pragma unroll
  for (int dt = 0; dt < C::DT; ++dt) oacc[dt][0] = oacc[dt][1] = zero4;
  // by query tile: softmax reference (log2 domain) and this lane's partial row sum
  float mref[2] = {0.f, 0.f}, lpart[2] = {0.f, 0.f};
  float done_m[2] = {0.f, 0.f}, done_l[2] = {0.f, 0.f};      // (VH) those of the item whose last P V product is under way

  // Epilogue of one item: O = R_n * acc / l + C_n (video rows; text rows: acc / l), bf16; then the
  // running state starts over for the next item. R_n and C_n are requested with the next
  // query rows: lane j holds elements CV*j .. CV*j+CV-1 of C_n, and every
  // lane reads the 64 it needs from LDS, 16 bytes at a time and all of a half of the channels before the first is used (one
  // word at a time through the crossbar, eight before a wait: with products of 32 x 32 x 16 506.6 us and 501.8 with it as it is,
  // 24 heads of 159 blocks, lists of 16; 15366 and 15247 with 931 and 94) -- no memory latency is left in here.
  constexpr int CV = D / 64;
  float done_comp[CV], next_comp[CV];            // of the item whose output is to be written; of the current one
#pragma unroll
  for (int j = 0; j < CV; ++j) done_comp[j] = next_comp[j] = 0.f;
  float done_rfac = 1.0f, next_rfac = 1.0f;
  // The query rows of the next item, and R_n and C_n of this one: asked for in the softmax phase of the last step but one (of an
  // item of two steps: in its last). The same number of vector loads in any case (NREQ).
  constexpr int NREQ = 2 * C::KS + 1;
  auto request_switch = [&]() __attribute__((always_inline)) {
    load_q(qnext, nxt_valid ? nxt.qo_off : cur.qo_off, nxt_valid ? nxt.q_count : cur.q_count);
    const size_t vrow = (size_t)cur.bh * dm.n + cur.qb;        // row of the per-video-block tensors
    next_rfac = 1.0f;
    if (cur.has_list && (a.flags & RSA_RECTIFY_CRITICAL)) {
      typedef const float __attribute__((address_space(4))) * const_f32_t;    // scalar load
      next_rfac = ((const_f32_t)(uintptr_t)a.R)[vrow];
    }
    // (an item without C_n: any readable words)
    const bool has_comp = cur.has_list && (a.flags & RSA_COMPENSATE);
    typedef float comp_t __attribute__((ext_vector_type(2), aligned(4)));
    const float* crow = has_comp ? a.comp + vrow * D : reinterpret_cast<const float*>(a.Q);
    const float* cp = crow + (has_comp ? lane_now() * CV : 0);
    if constexpr (CV == 2) {
      const comp_t c = *reinterpret_cast<const comp_t*>(cp);
      next_comp[0] = c.x;
      next_comp[CV - 1] = c.y;
    } else {
      next_comp[0] = *cp;
    }
  };
  // The current item ends: what was asked for takes its place. The compiler waits for the loads it knows of where they are
  // copied here, down to none outstanding; as it does not see the tile requests, this drains those as well, the V^T rows that
  // no one needs for another step among them.
  auto settle_switch = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        qreg[ks][f] = qnext[ks][f];
        asm volatile("" : "+v"(qreg[ks][f]));
      }
#pragma unroll
    for (int j = 0; j < CV; ++j) {
      done_comp[j] = next_comp[j];
      asm volatile("" : "+v"(done_comp[j]));
    }
    done_rfac = next_rfac;
  };
  // A piece of a row: the accumulators, four channels of a row to a lane, at the places where merge_kernel reads them (runs
  // of 256 bytes: [wave][32 channels][8 of them][the four channels][row]), row sums and references.
  auto write_piece = [&]() __attribute__((always_inline)) {
    const int ln = lane_now();
    const int l16 = ln % 16, g4 = ln / 16;
    float* p = sc.pieces + (size_t)((wg % 8) * sc.pieces_per_queue + done_piece) * (BLK * D + 2 * BLK);
    floatx4* dst = reinterpret_cast<floatx4*>(p) + wave * (C::DT * 2 * 64) + (g4 / 2) * 64 + (g4 % 2) * 32 + l16;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt) dst[dt * 128 + 16 * f] = oacc[dt][f];
      const float lsum = column_sum(C::VH ? done_l[f] : lpart[f]);
      if (g4 == 0) {
        p[BLK * D + wave * 32 + 16 * f + l16] = lsum;
        p[BLK * D + BLK + wave * 32 + 16 * f + l16] = C::VH ? done_m[f] : mref[f];
      }
    }
  };
  Tile vt_next = {};          // (VH) the tile of step s+1 as M(s) prepared it: its V^T rows are requested in M(s+1)
  // The rows of O go out whole: an accumulator lane holds four channels of one row at a time, and stored like that
  // (8 bytes of 32 rows per instruction) an item kept the address unit of the CU busy for 16 x 32 lines and wave. So
  // half of the channels at a time is turned through LDS: the V^T stage whose tile was read in the MFMA phase just ended is
  // free here (its next tile is requested in the one to come), and a wave uses only the 1 KB pieces that its own requests
  // fill, so no other wave can get in the way. 16-byte chunk c of row r lies at chunk c ^ row_key(r).
  // (With products of 32 x 32 x 16: 24 heads of 159 blocks, lists of 16, layer 684 -> 680 us; 2 x 12 heads of 160, d = 64, 860 -> 848;
  // 24 heads of 1182 blocks of 64 11164 -> 11090; the longer the lists the less: 24 heads of 931, lists of 94, 17295 -> 17277.)
  constexpr int ROWB = D;                          // bytes of half a row
  constexpr int RCH = ROWB / 16, RPC = 1024 / ROWB;   // chunks of half a row, rows per piece
  static_assert(VOFF == 1 && C::VPW * 1024 == 32 * ROWB, "a wave's own pieces of a V^T stage hold half of its 32 rows");
  auto row_key = [](int r) __attribute__((always_inline)) { return (r / (256 / ROWB)) % RCH; };
  int vst = 0;                // V^T ring stage of the current step (s % VSTAGES)
  auto write_rows = [&]() __attribute__((always_inline)) {
    const int vfree = C::VH ? (vst + 1 >= VSTAGES ? 0 : vst + 1) : (vst == 0 ? VSTAGES - 1 : vst - 1);
    const uint32_t turn = ldsV_addr + vfree * (C::VBUF * 16);
    typedef u32x2 __attribute__((address_space(3))) lds_u32x2;
    typedef u32x4 __attribute__((address_space(3))) lds_u32x4;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef f32x4 __attribute__((address_space(3))) lds_f32x4;
    typedef float __attribute__((address_space(3))) lds_f32;
    typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(4)));
    const bool do_comp = done_sparse && (a.flags & RSA_COMPENSATE);
    const int q_count = done_q_count;
    const int ln = lane_now();
    const int l16 = ln % 16, g4 = ln / 16;         // (copies of their own: see lane_now)
    float lsum[2], fac[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      lsum[f] = column_sum(C::VH ? done_l[f] : lpart[f]);
      fac[f] = done_rfac / lsum[f];
    }
    static_assert(16 % (256 / ROWB * RCH) == 0, "rows 16 apart have the same key");
    const int wkey = row_key(l16);
    const uint32_t wbase = turn + (l16 / RPC) * V_LDS_PASS + (l16 % RPC) * ROWB + 8 * (g4 % 2);
    const int rsub = ln / RCH;                     // row of a piece that this lane stores
    // (rows of one block: 32-bit byte offsets from the block's first row)
    char* obase = reinterpret_cast<char*>(a.O + done_qo_off);
    const uint32_t row_bytes = (uint32_t)dm.st * 2u;
    const uint32_t ooff = (uint32_t)(wave * 32 + rsub) * row_bytes;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      // the elements of C_n that go with these accumulators (16 dt + 4 g4 + e): through the wave's first piece, which the
      // rows of O take next
      f32x4 cadd[C::DT / 2];
#pragma unroll
      for (int d2 = 0; d2 < C::DT / 2; ++d2) cadd[d2] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (do_comp) {
#pragma unroll
        for (int j = 0; j < CV; ++j) *(lds_f32*)(uintptr_t)(turn + (uint32_t)(ln * CV + j) * 4u) = done_comp[j];
        asm volatile("" ::: "memory");             // (LDS instructions of a wave run in order)
#pragma unroll
        for (int d2 = 0; d2 < C::DT / 2; ++d2)
          cadd[d2] = *(const lds_f32x4*)(uintptr_t)(turn + 16 * g4 + 64 * (half * (C::DT / 2) + d2));
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int d2 = 0; d2 < C::DT / 2; ++d2) {
        const int dt = half * (C::DT / 2) + d2;
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          float o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float c = cadd[d2][e];
            o[e] = fmaf(oacc[dt][f][e], fac[f], c);
          }
          u32x2 w;
          w.x = pack_bf16x2(o[0], o[1]);
          w.y = pack_bf16x2(o[2], o[3]);
          *(lds_u32x2*)(uintptr_t)(wbase + f * (16 / RPC) * V_LDS_PASS + (((2 * d2 + g4 / 2) ^ wkey) * 16)) = w;
        }
      }
      asm volatile("" ::: "memory");               // (LDS instructions of a wave run in order)
#pragma unroll
      for (int i = 0; i < C::VPW; ++i) {
        const int r = i * RPC + rsub;
        const u32x4 v = *(const lds_u32x4*)(uintptr_t)(turn + i * V_LDS_PASS + ln * 16);
        if (wave * 32 + r < q_count)
          *reinterpret_cast<u32x4_u*>(obase + (ooff + (uint32_t)(i * RPC) * row_bytes + half * ROWB +
                                               16 * ((ln % RCH) ^ row_key(r)))) = v;
      }
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const int q = wave * 32 + 16 * f + l16;
      if (q < q_count && a.lse && g4 == 0)
        a.lse[((size_t)done_bh * dm.t) + done_q_t0 + q] = ((C::VH ? done_m[f] : mref[f]) + log2f(lsum[f])) * 0.6931471805599453f;
    }
  };
  auto write_output = [&]() __attribute__((always_inline)) {
    settle_products<16>(oacc);
    if (done_piece >= 0) write_piece();
    else write_rows();
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt) oacc[dt][0] = oacc[dt][1] = zero4;
    if constexpr (!C::VH) {
      mref[0] = mref[1] = 0.f;
      lpart[0] = lpart[1] = 0.f;
    }
  };

  // Two groups of waves share every SIMD (wave w of group 0 and wave w of group 1). They run
  // the same sequence  [M(s) | barrier | V(s) | barrier] ...  one barrier apart, so that while
  // one group issues MFMAs the other does its softmax on the VALU. s counts the steps of all the
  // items of the group, one after the other without a gap:
  //   M(s): O^T += V^T P^T of step s-1 (HALVES: half of the channels, of the block before the one of step s), then
  //         S^T = K Q^T of step s: matrix instructions, the A operand of each pair read from LDS a few slots ahead (V^T
  //         tile of step s-1 from its ring stage (s-1) % 3, HALVES: of s-2; K tile of step s from stage s % 2). Between
  //         them go the requests for the K rows of tile s+1 (into stage (s+1) % 2) and the V^T rows of tile s+1 (into
  //         stage (s+1) % 3; HALVES: of tile s, into s % 3). In the softmax phase, the longer of the two, a request
  //         costs some 50 cycles, here ten (all in V(s): 2700 cycles a step, half and half 2500, all here 2400).
  //   V(s): in the first step of an item (HALVES: the second), the output of the item before it; read the first V^T
  //         operands of M(s+1); mask, online softmax -> P as bf16 B operands (VALU only); fetch the list entry of step
  //         s+2; in the last step but one of an item request the query rows of the next item; wait for the K rows of
  //         tile s+1
  // The barrier after V(s) publishes the K rows of tile s+1 to the group, the one after M(s+1) the V^T rows that M(s)
  // requested. A K stage is rewritten two steps after it was read, a V^T stage three steps after it was
  // filled: by then every wave of the group has passed
  // the barrier that follows its last read. Every item has an even number of steps (SPB = 2 per key block),
  // so the position inside a key block and the K stage both follow from the parity of s, which the unrolled
  // loop knows.
  // key block that the next new-block step opens: entry m_nxt_e of a list, or block m_nxt_j (>= 0) of a dense row
  int m_nxt_e = 0, m_nxt_j = 0;
  uint64_t nxt_Kbytes = 0, nxt_Vtbytes = 0;   // ... and the K rows and V^T tiles of its item, where that may be the next one
  int kvc_cur = BLK;      // valid keys in the block of the current step
  int kvc_nxt = BLK;
  auto group_barrier = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  floatx4 sacc[C::KT][2];     // (key tile, query tile)
  u32x4 pb[C::PPC][2];        // probabilities as bf16 B operands: (32 keys, query tile)
  u32x4 pbn[2];               // (VH) those of the first half of a key block, while pb still holds the block before it
#pragma unroll
  for (int pc = 0; pc < C::PPC; ++pc) pb[pc][0] = pb[pc][1] = u32x4{0u, 0u, 0u, 0u};
  pbn[0] = pbn[1] = u32x4{0u, 0u, 0u, 0u};

  // M(s) is one fixed sequence of NPV + NQK slots of two MFMAs: the P V product of step s-1, then K Q^T
  // of step s. A slot takes one A operand (16 bytes per lane of the V^T or K tile) with the B operands of both query
  // tiles, which change places from slot to slot, so that every instruction shares an operand with the one before it. The A
  // operand is read from LDS W slots ahead of its MFMAs into a ring of W registers, so that LDS latency stays behind MFMAs
  // that already have their operands; the first W operands of a phase are read at the start of the
  // softmax phase before it. The order is pinned slot by slot.
  constexpr int NPV = C::PPC * C::PDT, NQK = C::KS * C::KT, NSLOT = NPV + NQK;
  constexpr int W = MWIN;
  static_assert(NPV >= W && NQK >= W, "the operands read ahead of a phase all belong to its first product");
  static_assert(W - W / 2 <= 4, "the operand waits are written out for at most four reads left outstanding");
  bf16x8 ring[W];
#pragma unroll
  for (int i = 0; i < W; ++i) ring[i] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
  const u32x4* vcur[C::PPC];  // vread[] moved to the V^T stage whose P V product comes next
#pragma unroll
  for (int pc = 0; pc < C::PPC; ++pc) vcur[pc] = vread[pc];
  auto read_v_operand = [&](int slot) __attribute__((always_inline)) {      // slot < NPV
    const int pc = slot / C::PDT, dt = slot % C::PDT;
    ring[slot % W] = __builtin_bit_cast(bf16x8, vcur[pc][dt * 16 * C::VCPR]);
  };
  // the operands of the first W slots of the next MFMA phase
  auto read_ahead = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < W; ++j) read_v_operand(j);
  };
  constexpr float kAbove = 1.0995116e12f, kBelow = 9.0949470e-13f;        // 2^+-kLazyBits
  static_assert(kLazyBits == 40.0f, "kAbove and kBelow are 2^+-kLazyBits");
  // (VH) Probabilities that wait for a P V product when the reference moves up by k binades (references are whole numbers
  // here): k off the exponents of both bf16 numbers of a register; what would go below 2^-126 saturates at 0.
  auto scaled = [](u32x4 w, uint32_t k) __attribute__((always_inline)) {
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const u16x2 off = __builtin_bit_cast(u16x2, k * 0x00800080u);
    auto pair = [&](uint32_t u) __attribute__((always_inline)) {
      return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, u), off));
    };
    return u32x4{pair(w.x), pair(w.y), pair(w.z), pair(w.w)};
  };

  // Variants of the two phases, all compile-time:
  //   MFMA phase  QK: 0 = the last P V product of the group alone.  LAST: the step is the last of its item
  //               -- the tile of step s+1 may open the next item (that item's K and V^T).
  //   softmax phase  FIRST: first step of an item.  OUT: the output of the item before is written first, if that is still to be
  //               done (the first step; HALVES: the second, and the last, which is the second of an item of one key block);
  //               FETCH: 0 none (odd steps), 1 the next entry of the item's own list, 2 wherever step
  //               s+2 falls (own list, first entry of the next item, or the last entry once more);
  //               LAST: behind it the next item takes the place of the current one.
  // The steps in the middle of an item run the plain variants in a loop of their own, so that what
  // only the boundaries between items need stays out of its registers.
  auto m_phase = [&](auto stc, auto qkc, auto lastc) __attribute__((always_inline)) {
    constexpr int ST = decltype(stc)::value;          // s modulo 2: the K stage and the part of the key block
    constexpr bool do_qk = decltype(qkc)::value != 0, last_of_item = decltype(lastc)::value != 0;
    constexpr int PART_NEXT = (ST + 1) % C::SPB;
    constexpr int OPEN = PART_NEXT == 0 ? kOpenPieces : 0;
    constexpr int MLOADS = LPS;                       // requests of this phase: K rows of step s+1, V^T rows of s+1 (VH: of step s)
    constexpr int LAST = do_qk ? NSLOT : NPV;         // slots that hold MFMAs
    // What goes between the MFMAs: the addresses of the tile of step s+1, then the requests. Whether that
    // step opens a new key block (its list entry came in during V(s-1)) follows from the parity of s. A group whose last step this
    // is requests the tile of its last list entry once more, into a stage nobody reads again.
    constexpr int REQ = OPEN + kStepPieces, TASKS = do_qk ? REQ + MLOADS : 0;
    // Requests of the four waves meet in the CU's one address unit, 16 cycles for each: with room for it, one in two or three
    // slots behind the addresses. Where slots are fewer than that (blocks of 64, d = 64), all tasks spread evenly over the phase:
    // two to a slot from its start leave its end bare (us, attention, packed and spread: d = 128, blocks of 64, 24 heads of 1182
    // blocks 6826 and 6687, all of 317 4437 and 4259, 4 of 128, lists of 13, 41.0 and 40.5; d = 64, blocks of 64, all of 64 81.2 and 79.3).
    constexpr bool FEW = !do_qk || TASKS > LAST || (LAST - REQ) / MLOADS < 2;
    constexpr int GAP = FEW ? 1 : (LAST - REQ) / MLOADS > 3 ? 3 : (LAST - REQ) / MLOADS;
    constexpr int WB = W / 2;                         // operands are waited for WB at a time
    Tile nt = {};
    // The wave that feeds the matrix pipe goes first wherever the two waves of a SIMD compete for an
    // issue slot: without this the older wave of the two wins, and the MFMA phases of the younger
    // group run a fifth longer than those of the other.
    __builtin_amdgcn_s_setprio(3);
    __builtin_amdgcn_sched_barrier(0);
    auto task = [&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      const int vnext = vst + 1 >= VSTAGES ? 0 : vst + 1;
      if constexpr (k < OPEN) {
        open_piece(kc, m_nxt_j >= 0 ? m_nxt_j : m_nxt_e, last_of_item ? nxt_Kbytes : cur.Kbytes,
                   last_of_item ? nxt_Vtbytes : cur.Vtbytes);
      } else if constexpr (k < REQ) {
        step_piece(IntC<k - OPEN>{}, nt, IntC<PART_NEXT>{}, (ST + 1) % KSTAGES, vnext);
      } else if constexpr (k < TASKS) {
        if constexpr (C::VH && k - REQ >= C::KPW) issue_load(vt_next, IntC<k - REQ>{});
        else issue_load(nt, IntC<k - REQ>{});
      }
    };
    static_for<0, LAST>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      // The operands of slots i .. i+WB-1 have arrived once at most the reads behind them are
      // outstanding: one wait per WB slots, and none is needed in between.
      if constexpr (i % WB == 0) {
        constexpr int behind = (LAST - i - WB) < 0 ? 0 : ((LAST - i - WB) < (W - WB) ? (LAST - i - WB) : (W - WB));
        // vmcnt and expcnt fields at "no wait", lgkmcnt = behind
        __builtin_amdgcn_s_waitcnt(0xC07F | (behind << 8));
        __builtin_amdgcn_sched_barrier(0);
      }
      auto product = [&](auto fc) __attribute__((always_inline)) {
        constexpr int f = decltype(fc)::value;
        if constexpr (i < NPV) {
          constexpr int pc = i / C::PDT, dt = (C::VH ? ST * C::PDT : 0) + i % C::PDT;
          // (VH: the first half of a block's probabilities is in pbn for the first product, in pb for the second)
          const u32x4 p = C::VH && ST == 0 && pc == 0 ? pbn[f] : pb[pc][f];
          mfma_add(oacc[dt][f], ring[i % W], __builtin_bit_cast(bf16x8, p));
        } else {
          constexpr int q = i - NPV, k2 = q / C::KT, t = q % C::KT;
          if constexpr (k2 == 0) mfma_first(sacc[t][f], ring[i % W], qreg[k2][f]);
          else mfma_add(sacc[t][f], ring[i % W], qreg[k2][f]);
        }
      };
      product(IntC<i % 2>{});
      if constexpr (TASKS > 0) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FEW) {
          static_for<TASKS * i / LAST, TASKS * (i + 1) / LAST>(task);
        } else if constexpr (i < REQ) {
          task(ic);
        } else {
          if constexpr ((i - REQ) % GAP == 0) task(IntC<REQ + (i - REQ) / GAP>{});
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      product(IntC<1 - i % 2>{});
      // the ring entry this slot used takes the operand of slot i + W
      if constexpr (i + W < LAST) {
        constexpr int slot = i + W;
        if constexpr (slot < NPV) {
          read_v_operand(slot);
        } else {
          constexpr int q = slot - NPV, k2 = q / C::KT, t = q % C::KT;
          ring[slot % W] = __builtin_bit_cast(bf16x8, kread[k2][(ST % KSTAGES) * KBUF + (32 * (t / 2) + 8 * (t % 2)) * C::KCPR]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (do_qk) {
      if constexpr (C::VH) vt_next = nt;
      kvc_nxt = blk_count;
    }
    // the V^T rows requested in the MFMA phase before this one have landed: the softmax phase reads the first of them
    if (last_of_item && cur.ns > C::SPB) wait_loads_leaving<do_qk ? MLOADS + NREQ : 0>();
    else wait_loads_leaving<do_qk ? MLOADS : 0>();
  };

  // entry j of an item's list; a dense row: j itself
  auto list_entry = [&](const Item& it, int j) __attribute__((always_inline)) {
    const int e = it.list[it.has_list ? j : 0];
    return it.has_list ? e : span_first(it.span) + j;
  };

  int fj = 0;                 // entry of the current item's list that the next even step fetches
  int have_output = 0;        // an item has ended and its output is still in the accumulators
  auto v_phase = [&](auto stc, auto firstc, auto outc, auto fetchc, auto lastc) __attribute__((always_inline)) {
    constexpr int ST = decltype(stc)::value;
    constexpr bool first_of_item = decltype(firstc)::value != 0, last_of_item = decltype(lastc)::value != 0;
    constexpr bool output = decltype(outc)::value != 0;
    constexpr int FETCH = decltype(fetchc)::value;
    __builtin_amdgcn_s_setprio(0);
    constexpr int VLOADS = C::VPW;  // the last requests of M(s): V^T rows, which may still be out when this phase ends
    // The last step of an item asks for the entry of the item after the one after the next.
    Entry entry_new = {};
    bool more = false;
    if constexpr (C::VH && first_of_item) {
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        done_m[f] = mref[f];
        done_l[f] = lpart[f];
        mref[f] = lpart[f] = 0.f;
      }
    }
    const bool had_output = have_output;
    if constexpr (C::VH && output) {               // (ahead of what the last step of an item of one key block asks for)
      if (have_output) {
        __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
        write_output();
        have_output = 0;
      }
    }
    if constexpr (last_of_item) {
      if (cur.ns == C::SPB) request_switch();
      more = k_next < n_my_items;
      if (k_next + 1 < n_my_items) entry_new = my_entry(k_next + 1);
    }
    // The list entry of step s+2 (an even step opens a key block) for M(s+1): requested ahead of the
    // softmax, which hides the scalar cache miss that every sixteenth entry (and the head of every list)
    // is. Only the load is here -- what the entry means (a dense row has none: its j-th block is j)
    // is settled where M(s+1) opens the block.
    if constexpr (FETCH == 1) {
      m_nxt_e = cur.list[cur.has_list ? fj : 0];
      m_nxt_j = cur.has_list ? -1 : span_first(cur.span) + fj;
      fj += 1;
    } else if constexpr (FETCH == 2) {
      // it may be the first entry of the next item; past the last item, the last entry again (a valid
      // block: the tile requested for a step that does not exist is never read)
      const int nlist = span_len(cur.span);
      const bool own = fj < nlist, follow = !own && nxt_valid;
      const_list_t lp = follow ? nxt.list : cur.list;
      const int hl = follow ? nxt.has_list : cur.has_list;
      const int j = own ? fj : (follow ? 0 : nlist - 1);
      nxt_Kbytes = follow ? nxt.Kbytes : cur.Kbytes;
      nxt_Vtbytes = follow ? nxt.Vtbytes : cur.Vtbytes;
      m_nxt_e = lp[hl ? j : 0];
      m_nxt_j = hl ? -1 : span_first(follow ? nxt.span : cur.span) + j;
      fj += 1;
    }
    // Step ns-2 of an item of two key blocks or more; an item of one block asks in its last phase instead (a request under a
    // condition in the first phase would leave the compiler with loads that may be pending on its way into the loop of steps,
    // and with a wait for them in every other step).
    constexpr bool requests = FETCH == 2 && !first_of_item;
    // the first step of an item: the P V products of the item before it are complete
    // (the K rows of tile s+1 are waited for first: at the end of the phase the stores would be waited for with them,
    // which now complete under the next MFMA phase)
    if constexpr (!C::VH && output) {
      if (have_output) {
        wait_loads_leaving<VLOADS>();
        write_output();
      }
    }
    // the first V^T operands of M(s+1), from the stage of this step (VH: of the step before), published before the barrier
    // that this phase began with
    const int vst_read = !C::VH ? vst : vst == 0 ? VSTAGES - 1 : vst - 1;
#pragma unroll
    for (int pc = 0; pc < C::PPC; ++pc) vcur[pc] = vread[pc] + vst_read * C::VBUF;
    read_ahead();
    __builtin_amdgcn_sched_barrier(0);
    float rs[2];
    // The scores go through in a line, the two query tiles together: multiplied and taken from the reference, two places on
    // to the exponential, two further on to the sum and the conversion. Beside the other group's products the vector
    // ALU takes two instructions (one exponential) for each of them, and an instruction whose operand has only just been asked
    // for takes as long as two that wait for nothing (left to the compiler, which chained them: 150 cycles more). With the 16
    // scores of a lane that a step of a block of 64 has, and the products of d = 128 beside them, the compiler's own order is the
    // better one (us, attention, in a line and its own: 4 heads of 128 blocks, lists of 13, 40.6 and 40.1; 4 of 19, lists of 8, 29.1
    // and 28.7; 24 of 1182 6685 and 6664; d = 64, 24 of 317 346.6 and 349.1, all of 64 blocks 79.3 and 80.1).
    constexpr bool IN_LINE = C::KT > 2 || D == 64;
    auto probabilities = [&]() __attribute__((always_inline)) {
      constexpr int NE = 16 * C::PC, LAG = 2;
      float x[NE], p[NE];
      uint32_t w[NE / 2];
      static_for<0, NE / 2 + 2 * LAG>([&](auto ec) __attribute__((always_inline)) {
        constexpr int e = 2 * decltype(ec)::value, E = e - 2 * LAG, A = e - 4 * LAG;
        if constexpr (e < NE) {
          constexpr int j = e / 16, i = e / 2 % 8;
#pragma unroll
          for (int f = 0; f < 2; ++f) x[e + f] = fmaf(sacc[2 * j + i / 4][f][i % 4], cs, -mref[f]);
        }
        if constexpr (E >= 0 && E < NE) {
#pragma unroll
          for (int f = 0; f < 2; ++f) p[E + f] = __builtin_amdgcn_exp2f(x[E + f]);
        }
        if constexpr (A >= 0) {
          constexpr int j = A / 16, i = A / 2 % 8;
#pragma unroll
          for (int f = 0; f < 2; ++f) rs[f] = A == 0 ? p[f] : rs[f] + p[A + f];
          if constexpr (i % 2 == 1) {
#pragma unroll
            for (int f = 0; f < 2; ++f) {
              uint32_t u = pack_bf16x2(p[A - 2 + f], p[A + f]);
              asm volatile("" : "+v"(u));          // (here, and not behind the branch that may want it otherwise)
              w[8 * j + 4 * f + i / 2] = u;
            }
          }
        }
        if constexpr (IN_LINE) __builtin_amdgcn_sched_barrier(0);
      });
#pragma unroll
      for (int j = 0; j < C::PC; ++j)
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          const u32x4 v = {w[8 * j + 4 * f], w[8 * j + 4 * f + 1], w[8 * j + 4 * f + 2], w[8 * j + 4 * f + 3]};
          if constexpr (!C::VH) pb[j][f] = v;
          else if constexpr (ST == 0) pbn[f] = v;
          else pb[1][f] = v;
        }
    };
    {
      const int kv_count = kvc_cur;
      // (the first scores taken are those of tiles 0 and 1, whose last products four others followed where there are more tiles;
      // those of the other tiles are taken far enough down the line)
      settle_products<(C::KT > 2 ? 1 : 8)>(sacc);
      // accumulator register r of key tile t is key part*KVS + 32(t/2) + 8(t%2) + r + key_row(4*g4) of the block
      // (rare, like the branch below: out of line, the path that every step takes has no jump over it)
      if (__builtin_expect(kv_count < BLK, 0)) {
        // (constants against one lane-dependent bound: compared the other way round, the key numbers are 32 registers that
        // the compiler keeps through the whole loop)
        int valid = kv_count - (ST % C::SPB) * KVS - key_row(4 * g4);
        // (here the compiler takes the tiles in any order: the last products are waited for ahead of the first comparison)
        asm volatile("s_nop 7" : "+v"(valid));
#pragma unroll
        for (int t = 0; t < C::KT; ++t)
#pragma unroll
          for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (32 * (t / 2) + 8 * (t % 2) + r >= valid) sacc[t][f][r] = -INFINITY;
      }
      // ---- online softmax, two query columns per lane, one of each query tile ---------------------------------
      // Scores are counted in binades (score * scale * log2 e) from a reference that starts at 0 for
      // every item and moves rarely: fp32 sums and bf16 operands span 2^+-126, so probabilities may
      // sit anywhere within 2^+-kLazyBits of one another's scale. No maximum is taken on the way: the
      // probabilities of the step are worked out against the current reference, and only when their
      // sum says that one of them left the window (above it; in the first step of an item, all of
      // them below it, too) is the step done again the long way -- the scores are still in registers
      // -- with the row maximum as the new reference and everything gathered so far rescaled.
      if constexpr (C::VH && ST == 0) {
        pb[0][0] = pbn[0];
        pb[0][1] = pbn[1];
      }
      probabilities();
      float largest;             // (fmaxf would put two more instructions into this chain, to quiet signalling NaNs)
      asm("v_max_f32 %0, %1, %2" : "=v"(largest) : "v"(rs[0]), "v"(rs[1]));
      bool outside = largest > kAbove;
      if constexpr (first_of_item) outside = outside || rs[0] < kBelow || rs[1] < kBelow;
      if (__builtin_expect(__any(outside), 0)) {
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          float mx = -INFINITY;
#pragma unroll
          for (int t = 0; t < C::KT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sacc[t][f][r]);
          mx = column_max(mx) * cs;                      // the scale is positive
          if constexpr (C::VH) mx = ceilf(mx);           // probabilities that wait are rescaled as they are: by powers of two
          if constexpr (first_of_item) {
            // Accumulators and row sum are empty: nothing to rescale. Scores that are all -inf (keys that mask
            // themselves) must not become the reference, -inf - -inf is no number: below the lowest finite one their
            // probabilities are 0, and the first finite score leaves the window and brings its own reference.
            mref[f] = fmaxf(mx, -3.4028234663852886e38f);
          } else {
            const float mnew = fmaxf(mref[f], mx);
            const float alpha = __builtin_amdgcn_exp2f(mref[f] - mnew);
            const float before = mref[f];
            mref[f] = mnew;
            lpart[f] *= alpha;
            if constexpr (!(C::VH && output && !last_of_item)) {     // (there they have just been emptied)
#pragma unroll
              for (int dt = 0; dt < C::DT; ++dt) {
                floatx4 o = oacc[dt][f];
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] *= alpha;
                asm volatile("" : "+v"(o));      // (or the accumulators are copied between registers in every phase)
                oacc[dt][f] = o;
              }
            }
            if constexpr (C::VH) {
              const uint32_t up = (uint32_t)fminf(mref[f] - before, 255.f);
              if constexpr (ST == 1) {
                u32x4 w = scaled(pbn[f], up);
                asm volatile("" : "+v"(w));      // (or the accumulators are copied between registers in every MFMA phase)
                pbn[f] = w;
              } else {
#pragma unroll
                for (int pc = 0; pc < C::PPC; ++pc) pb[pc][f] = scaled(pb[pc][f], up);
              }
            }
          }
        }
        probabilities();
      }
      lpart[0] += rs[0];
      lpart[1] += rs[1];
    }
    if constexpr (requests) request_switch();
    kvc_cur = kvc_nxt;
    // the probabilities are complete here: nothing of the softmax may sink behind the barrier
    // into the MFMA phase, where it would take the other group's VALU time
#pragma unroll
    for (int pc = 0; pc < C::PPC; ++pc) asm volatile("" : "+v"(pb[pc][0]), "+v"(pb[pc][1]));
    if constexpr (C::VH) asm volatile("" : "+v"(pbn[0]), "+v"(pbn[1]));
    // (the list entry is waited for here, where nothing else is under way, and not in M(s+1) together with its operands)
    if constexpr (FETCH != 0) asm volatile("" : "+s"(m_nxt_e));
    asm volatile("" : "+v"(lpart[0]), "+v"(mref[0]), "+v"(lpart[1]), "+v"(mref[1]));
    vst = vst + 1 >= VSTAGES ? 0 : vst + 1;
    if constexpr (last_of_item) {
      // the item has ended: its output waits for the last P V product; the next item takes its place
      done_bh = cur.bh;
      done_sparse = cur.has_list;
      done_q_t0 = cur.q_t0;
      done_q_count = cur.q_count;
      done_qo_off = cur.qo_off;
      done_piece = (cur.span & kSpanPartial) ? next_piece++ : -1;
      have_output = 1;
      if (nxt_valid) {
        cur = nxt;
        fj = 1;                          // entry 0 was fetched two steps ago
        nxt_valid = more;
        if (more) nxt = make_item(ahead);
        ahead = entry_new;
        k_next += 1;
      }
    }
    // the K rows of tile s+1 have landed (this wave's share; the barrier that follows covers the group; loads return in order:
    // only the V^T rows behind them and this phase's own requests may still be out)
    // (VH: behind the last step of all there is no other phase to wait for its V^T rows)
    constexpr int LEAVING = C::VH && last_of_item ? 0 : VLOADS + (requests ? NREQ : 0);
    if constexpr (output) {
      if (!had_output) wait_loads_leaving<LEAVING>();
    } else {
      wait_loads_leaving<LEAVING>();
    }
    if constexpr (last_of_item) settle_switch();
    group_barrier();
  };

  const bool active = n_my_items > 0;
  if (active) {
    cur = load_item(0);
    nxt_valid = n_my_items > 1;
    if (nxt_valid) nxt = load_item(1);
    k_next = 2;
    if (n_my_items > 2) ahead = my_entry(2);
    load_q(qreg, cur.qo_off, cur.q_count);
    Tile t0;
    const int m0 = list_entry(cur, 0);
    static_for<0, kOpenPieces>([&](auto pc) __attribute__((always_inline)) { open_piece(pc, m0, cur.Kbytes, cur.Vtbytes); });
    static_for<0, kStepPieces>([&](auto pc) __attribute__((always_inline)) { step_piece(pc, t0, IntC<0>{}, 0, 0); });
    static_for<0, (C::VH ? C::KPW : LPS)>([&](auto ic) __attribute__((always_inline)) { issue_load(t0, ic); });
    if constexpr (C::VH) vt_next = t0;
    // The compiler does not see the direct-to-LDS loads: it has to place its wait for Q here, not at the first use inside
    // the loop, where it would be a wait for every load outstanding.
    __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) asm volatile("" : "+v"(qreg[ks][0]), "+v"(qreg[ks][1]));
    kvc_cur = blk_count;
    fj = 1;
    // The first MFMA phase (VH: the first two) multiplies the (zero) probabilities of a step that does not exist with
    // whatever the last V^T stage (VH: the last two) holds: make that zeros too (0 x NaN would poison the accumulators).
    {
      constexpr int FROM = C::VH ? VSTAGES - 2 : VSTAGES - 1;
      u32x4* vlast = lds + KSTAGES * KBUF + FROM * C::VBUF;
      for (int c = wave * 64 + lane; c < (VSTAGES - FROM) * C::VBUF; c += C::NW * 64) vlast[c] = u32x4{0u, 0u, 0u, 0u};
      // ... and the operands read ahead of it come from there
#pragma unroll
      for (int pc = 0; pc < C::PPC; ++pc) vcur[pc] = vread[pc] + FROM * C::VBUF;
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0070);
  group_barrier();                  // tile 0 of every group is in LDS
  if (active) read_ahead();
  if (grp >= NGRP / 2) group_barrier();    // the second half of the groups runs one barrier behind the first
  // Every group turns wg_rounds rounds of two barriers; round s is M(s), V(s) while the group has
  // steps left, the last P V product and the last output in round my_total, and nothing but the
  // barriers after.
  using Y = IntC<1>;
  using N = IntC<0>;
  int s = 0;
  if (active) {
    for (int item = 0; item < n_my_items; ++item) {
      const int ns = cur.ns;
      // step 0 of the item
      m_phase(IntC<0>{}, Y{}, N{});
      group_barrier();
      v_phase(IntC<0>{}, Y{}, IntC<C::VH ? 0 : 1>{}, IntC<2>{}, N{});
      if constexpr (C::VH) {
        if (ns >= 4) {
          // step 1 writes the output of the item before
          m_phase(IntC<1>{}, Y{}, N{});
          group_barrier();
          v_phase(IntC<1>{}, N{}, Y{}, IntC<0>{}, N{});
          // steps 2 .. ns-3 in pairs
          for (int sj = 2; sj + 2 < ns; sj += 2) {
            m_phase(IntC<0>{}, Y{}, N{});
            group_barrier();
            v_phase(IntC<0>{}, N{}, N{}, IntC<1>{}, N{});
            m_phase(IntC<1>{}, Y{}, N{});
            group_barrier();
            v_phase(IntC<1>{}, N{}, N{}, IntC<0>{}, N{});
          }
          // step ns-2 fetches the first list entry of the next item
          m_phase(IntC<0>{}, Y{}, N{});
          group_barrier();
          v_phase(IntC<0>{}, N{}, N{}, IntC<2>{}, N{});
        }
        // step ns-1 (of an item of one key block: step 1, with the output of the item before)
        m_phase(IntC<1>{}, Y{}, Y{});
        group_barrier();
        v_phase(IntC<1>{}, N{}, Y{}, IntC<0>{}, Y{});
      } else {
        if (ns >= 4) {
          // steps 1 .. ns-4 in pairs: nothing but this item's own list and tiles
          for (int sj = 1; sj + 3 < ns; sj += 2) {
            m_phase(IntC<1>{}, Y{}, N{});
            group_barrier();
            v_phase(IntC<1>{}, N{}, N{}, IntC<0>{}, N{});
            m_phase(IntC<0>{}, Y{}, N{});
            group_barrier();
            v_phase(IntC<0>{}, N{}, N{}, IntC<1>{}, N{});
          }
          // steps ns-3 and ns-2: the latter fetches the first list entry of the next item
          m_phase(IntC<1>{}, Y{}, N{});
          group_barrier();
          v_phase(IntC<1>{}, N{}, N{}, IntC<0>{}, N{});
          m_phase(IntC<0>{}, Y{}, N{});
          group_barrier();
          v_phase(IntC<0>{}, N{}, N{}, IntC<2>{}, N{});
        }
        // step ns-1
        m_phase(IntC<1>{}, Y{}, Y{});
        group_barrier();
        v_phase(IntC<1>{}, N{}, N{}, IntC<0>{}, Y{});
      }
      s += ns;
    }
    m_phase(IntC<0>{}, N{}, N{});
    if constexpr (C::VH) {
      // the second half of the channels (its V^T tile was published a step ago)
      pb[0][0] = pbn[0];
      pb[0][1] = pbn[1];
      const int vst_read = vst == 0 ? VSTAGES - 1 : vst - 1;
#pragma unroll
      for (int pc = 0; pc < C::PPC; ++pc) vcur[pc] = vread[pc] + vst_read * C::VBUF;
      read_ahead();
      m_phase(IntC<1>{}, N{}, N{});
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        done_m[f] = mref[f];
        done_l[f] = lpart[f];
      }
    }
    group_barrier();
    __builtin_amdgcn_s_setprio(0);
    write_output();
    // nothing may be in flight into the LDS of a workgroup that is about to end
    __builtin_amdgcn_s_waitcnt(0x0F70);
    group_barrier();
    s += 1;
  }
  for (; s < wg_rounds; ++s) {
    group_barrier();
    group_barrier();
  }
  if (grp < NGRP / 2) group_barrier();
}

// Where the schedule's parts lie in the room it is given (bytes from its start, all 256-byte aligned).
struct SchedLayout {
  size_t nitems, total, piece0, cross, info, table, schedule, pieces, bytes;
};
SchedLayout sched_layout(const Dims& dm, const SchedShape& sh) {
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t slots = (size_t)kQueues * sh.slots, pieces = (size_t)kQueues * sh.pieces_per_queue;
  SchedLayout l;
  size_t off = 0;
  l.nitems = off;  off += up(slots * sizeof(int32_t));
  l.total = off;   off += up(slots * sizeof(int32_t));
  l.piece0 = off;  off += up(slots * sizeof(int32_t));
  l.cross = off;   off += up(kQueues * kQueues * sizeof(int2));
  l.info = off;    off += up(pieces * sizeof(int2));
  l.table = off;   off += up(slots * sh.cap * sizeof(int2));
  l.schedule = off;
  l.pieces = off;  off += pieces * piece_floats(dm.d, dm.blk) * sizeof(float);
  l.bytes = off;
  return l;
}

template <int D, int BLK, bool HALVES>
hipError_t launch_attn_t(const Dims& dm, const AttnArgs& a, const AttnSched& ws, hipStream_t s) {
  using C = AttnCfg<D, BLK, HALVES>;
  const bool dense_all = (a.flags & RSA_DENSE) != 0;
  const int n_wg = ws.n_wg;
  if (n_wg < 8 || n_wg % 8) return hipErrorInvalidValue;
  SchedShape sh = sched_shape(dm, a.flags, n_wg, C::NGRP);
  SchedArgs sc = {};
  sc.n_items = sh.n_items;
  sc.n_dense = dense_all ? sh.n_items : sh.n_dense;
  sc.dense_per_bh = dense_all ? dm.m : (dm.mt > 0 ? dm.mt : 1);
  sc.dense_first = dense_all ? 0 : dm.n;
  const bool compensate = !dense_all && (a.flags & RSA_COMPENSATE);
  SchedLayout l = sched_layout(dm, sh);
  if (l.bytes > ws.room_bytes) {                   // no room for pieces: nothing is cut
    sh.pieces_per_queue = sh.n_cross = 0;
    l = sched_layout(dm, sh);
  }
  if (l.bytes > ws.room_bytes) {                   // nor for the whole table: fewer entries per slot, down to the average share
    const size_t entry = (size_t)kQueues * sh.slots * sizeof(int2), over = (l.bytes - ws.room_bytes + entry - 1) / entry;
    sh.cap -= (int)(over < (size_t)(sh.cap - sh.least_cap) ? over : (size_t)(sh.cap - sh.least_cap));
    l = sched_layout(dm, sh);
  }
  const bool deal = ws.room && l.bytes <= ws.room_bytes && sh.slots <= kMaxSlots;
  DealArgs da = {};
  if (deal) {
    char* room = (char*)ws.room;
    da.table = (int2*)(room + l.table);
    da.nitems = (int32_t*)(room + l.nitems);
    da.total = (int32_t*)(room + l.total);
    da.piece0 = (int32_t*)(room + l.piece0);
    da.piece_info = (int2*)(room + l.info);
    da.cross = (int2*)(room + l.cross);
    da.pieces = (float*)(room + l.pieces);
    da.cap = sh.cap; da.slots = sh.slots; da.groups = C::NGRP; da.pieces_per_queue = sh.pieces_per_queue;
    da.heads_at_once = sh.heads_at_once; da.most_share = sh.most_share; da.rows_per_bh = sh.rows_per_bh;
    da.n_dense = sh.n_dense; da.dense_per_bh = sh.dense_per_bh > 0 ? sh.dense_per_bh : 1;
    da.dense_first = sh.dense_first; da.n_cross = sh.n_cross; da.min_piece = sh.min_piece; da.switch_cost = sh.switch_cost;
    da.rule = cut_rule(dm);
    sc.table = da.table; sc.nitems = da.nitems; sc.total = da.total; sc.piece0 = da.piece0; sc.pieces = da.pieces;
    sc.cap = sh.cap; sc.slots_per_queue = sh.slots; sc.pieces_per_queue = sh.pieces_per_queue;
  }
  // With no more items than slots every row starts at once: no order helps, and the launch is saved.
  AttnArgs aa = a;
  if (sh.n_items <= kQueues * sh.slots) aa.row_order = nullptr;
  const hipError_t side = launch_attn_side(dm, aa, da, !dense_all && aa.row_order && deal, compensate, deal, s);
  if (side != hipSuccess) return side;
  hipLaunchKernelGGL((attn_kernel<D, BLK, HALVES>), dim3((unsigned)n_wg), dim3(C::NTHR), 0, s, dm, aa, sc);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !deal || sh.pieces_per_queue == 0) return e;
  return launch_attn_merge(dm, aa, da, s);
}

}  // namespace

// The larger of what a sparse and a dense launch on RSA_ATTN_MAX_WGS resident workgroups need. (A GPU
// with fewer CUs has fewer, longer queues; should its table not fit, the items go out in index order.)
void attn_sched_bytes(const Dims& dm, size_t* schedule, size_t* pieces) {
  *schedule = *pieces = 0;
  for (int flags : {0, (int)RSA_DENSE}) {
    const SchedLayout l = sched_layout(dm, sched_shape(dm, flags, RSA_ATTN_MAX_WGS, dm.blk == 128 ? 2 : 4));
    *schedule = l.schedule > *schedule ? l.schedule : *schedule;
    *pieces = l.bytes - l.schedule > *pieces ? l.bytes - l.schedule : *pieces;
  }
}

hipError_t launch_attn(const Dims& dm, const AttnArgs& a, const AttnSched& ws, hipStream_t s) {
  if (dm.d == 128 && dm.blk == 128) return launch_attn_t<128, 128, false>(dm, a, ws, s);
  if (dm.d == 128 && dm.blk == 64 && !(a.flags & RSA_DENSE)) return launch_attn_t<128, 64, true>(dm, a, ws, s);   // (HALVES)
  if (dm.d == 128 && dm.blk == 64) return launch_attn_t<128, 64, false>(dm, a, ws, s);
  if (dm.d == 64 && dm.blk == 128) return launch_attn_t<64, 128, false>(dm, a, ws, s);
  return launch_attn_t<64, 64, false>(dm, a, ws, s);
}

}  // namespace rsa
