// The small kernels around the persistent attention kernel (paper Alg. 1 step 21 for the pooled
// compensation; the launch order and the schedule are this library's own): row_rank_kernel,
// compensation_kernel, schedule_kernel, and compensation_schedule_kernel = the second and the third in one
// launch, before it; merge_kernel behind it when rows were cut.
#include "attn_sched.hpp"

namespace rsa {
namespace {

// Pooled compensation (Alg. 1 step 21): C[n][:] = sum over blocks m that are not kept and
// have their M_c bit set of A^pool[n][m] * v^pool[m][:], all fp32. Written as the product it is:
// W V^pool with W[n][m] = A^pool[n][m] where block m is compensated for row n and 0 elsewhere
// (about a fifth of the entries at the benchmark shape), on v_mfma_f32_32x32x2_f32 -- fp32 operands,
// fp32 products and sums. One workgroup per 32 query blocks of a (batch, head); the key blocks come
// 64 at a time: the weights of the 32 rows (read whole, masked on their way into LDS) and the 64 rows
// of v^pool go through LDS, the next 64 are on their way while
// the matrix instructions of these run; wave w owns channels 32 w .. 32 w + 31 (M = query row,
// N = channel, k = key block: the lower half-wave takes blocks 8u .. 8u+3 of a run of eight, the
// upper one 8u+4 .. 8u+7, both operands alike). Blocks past the end of the row carry weight 0.
// v^pool of a head is read once per workgroup (from L2) instead of once per compensated pair.
// Four workgroups fit a CU (40 KB of LDS, 97 registers): 24 heads of 1182 blocks 154 -> 121 us against three.
constexpr int kCompChunk = 64;                   // key blocks per pass
template <int D>
constexpr unsigned comp_lds_bytes() { return (32 * kCompChunk + kCompChunk * D) * 4; }
// 16-byte chunk c of row r of the weight tile sits at chunk position c ^ r % 16: sixteen rows read at one chunk index touch
// every bank once. (Padded rows did too, but then only three workgroups fit a CU: 24 heads of 1182 blocks, 888 workgroups,
// took a second round on 768 places.)
__device__ __forceinline__ int comp_weight_at(int r, int c) { return r * kCompChunk + 4 * (c ^ (r & 15)); }
static_assert(kCompChunk == 64, "sixteen chunks to a row");

template <int D>
__device__ __forceinline__ void compensate_tile(const Dims& dm, const AttnArgs& a, int n0, int bh, uint32_t* lds) {
  constexpr int MC = kCompChunk;
  constexpr int CT = D / 32;                     // channel tiles = waves with matrix work
  constexpr int VL = MC * D / 4 / 256;           // 16-byte loads of v^pool per thread and pass
  float* wt = reinterpret_cast<float*>(lds);     // [32][MC], comp_weight_at
  float* vt = wt + 32 * MC;                      // [MC][D]
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, l32 = lane % 32, hf = lane / 32;
  const float* Vp = a.Vp + (size_t)bh * dm.m * D;
  // this thread's share of the weight tile: row tid / 8, the eight blocks from 8 (tid % 8) on (one mask word)
  const int wr = tid / 8, wc = (tid % 8) * 8;
  const bool row_ok = n0 + wr < dm.n;
  const size_t row = (size_t)bh * dm.n + (row_ok ? n0 + wr : dm.n - 1);
  const uint32_t* kept = a.mask_bits + row * dm.w;
  const uint32_t* gate = a.Mc_bits + row * dm.w;
  const float* A = a.Apool + row * dm.m;
  float w[8];
  uint32_t on = 0u;                              // bits of this thread's eight blocks: compensated or not
  floatx4 vv[VL];
  typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));     // rows of A^pool start at any word
  // Nothing here depends on anything else loaded here: the weights are read whole and masked when they go to LDS.
  auto fetch = [&](int m0) __attribute__((always_inline)) {
    const int m = m0 + wc;
    on = 0u;
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = 0.f;
    if (row_ok && m < dm.m) {
      on = (~kept[m / 32] & gate[m / 32]) >> (m % 32);
      if (m + 8 <= dm.m) {
        const floatx4 lo = *reinterpret_cast<const floatx4_u*>(A + m), hi = *reinterpret_cast<const floatx4_u*>(A + m + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { w[e] = lo[e]; w[4 + e] = hi[e]; }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) if (m + e < dm.m) w[e] = A[m + e];
      }
    }
#pragma unroll
    for (int i = 0; i < VL; ++i) {
      const int idx = tid + 256 * i, r = idx / (D / 4), c4 = idx % (D / 4);
      const int mm = m0 + r < dm.m ? m0 + r : dm.m - 1;        // rows past the end repeat the last one (weight 0)
      vv[i] = *reinterpret_cast<const floatx4*>(Vp + (size_t)mm * D + 4 * c4);
    }
  };
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  fetch(0);
  for (int m0 = 0; m0 < dm.m; m0 += MC) {
    __syncthreads();                             // the tiles of the pass before have been read
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = ((on >> e) & 1u) ? w[e] : 0.f;
    *reinterpret_cast<floatx4*>(wt + comp_weight_at(wr, wc / 4)) = floatx4{w[0], w[1], w[2], w[3]};
    *reinterpret_cast<floatx4*>(wt + comp_weight_at(wr, wc / 4 + 1)) = floatx4{w[4], w[5], w[6], w[7]};
#pragma unroll
    for (int i = 0; i < VL; ++i) {
      const int idx = tid + 256 * i;
      *reinterpret_cast<floatx4*>(vt + 4 * idx) = vv[i];      // row idx / (D/4), chunk idx % (D/4): rows are D floats
    }
    __syncthreads();
    if (m0 + MC < dm.m) fetch(m0 + MC);
    if (wave < CT) {
#pragma unroll
      for (int u = 0; u < MC / 8; ++u) {
        const floatx4 a4 = *reinterpret_cast<const floatx4*>(wt + comp_weight_at(l32, 2 * u + hf));
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[e], vt[(8 * u + 4 * hf + e) * D + 32 * wave + l32], acc, 0, 0, 0);
      }
    }
  }
  // accumulator register r: query block n0 + 8(r/4) + 4*hf + r%4, channel 32*wave + l32
  if (wave < CT) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int n = n0 + 8 * (r / 4) + 4 * hf + (r % 4);
      if (n < dm.n) a.comp[((size_t)bh * dm.n + n) * D + 32 * wave + l32] = acc[r];
    }
  }
}

template <int D>
__global__ __launch_bounds__(256) void compensation_kernel(Dims dm, AttnArgs a) {
  extern __shared__ uint32_t side_lds[];
  compensate_tile<D>(dm, a, blockIdx.x * 32, blockIdx.y, side_lds);
}

// Launch order of the video query blocks of one (batch, head): sorted by their first three
// kept key blocks (ties: block index). Groups of waves that are resident on an XCD at the same time
// then walk similar lists and find each other's K/V tiles in that XCD's L2 (on the benchmark
// inputs the traffic that crosses the fabric drops by 40 %). A heuristic: any permutation gives
// the same results. The keys are distinct (the block index is part of them), so the place of a row is the
// number of smaller keys: a workgroup gathers the keys of a head in LDS and counts for 64 of its rows, four
// threads to a row. One workgroup per head sorting the keys took 21 us at 929 rows (24 heads) and 12 us at 159,
// most of it barriers of a chip that stood still; counting takes 11 and 5 us, the gathering of the keys (a cache
// line per row, in every workgroup) being most of it.
// An entry of the order: the row, and the load (key blocks and switches) of the rows before it, in units of 32 key blocks
// (at most 4095 (4096 + 6) / 32 < 2^20).
constexpr int kRankRows = 64;
__device__ __forceinline__ int32_t order_entry(int row, int load) {
  return (int32_t)((uint32_t)row | (uint32_t)(load / 32) << 12);
}
__device__ __forceinline__ int order_row(int32_t entry) { return entry & 4095; }
__device__ __forceinline__ int order_load(int32_t entry) { return (int)((uint32_t)entry >> 12); }
__global__ __launch_bounds__(256) void row_rank_kernel(Dims dm, AttnArgs a, int switch_cost) {
  __shared__ uint64_t keys[RSA_MAX_BLOCKS + 32];
  const int bh = blockIdx.y, tid = threadIdx.x;
  const int padded = (dm.n + 31) & ~31;                     // the counting loop takes 32 keys at a time
  const int e1 = min(1, dm.m - 1), e2 = min(2, dm.m - 1);
#pragma unroll 4
  for (int i = tid; i < padded; i += 256) {
    const int r = min(i, dm.n - 1);
    const size_t row = (size_t)bh * dm.n + r;
    const int cnt = a.count[row];
    const int32_t* lst = a.block_idx + row * dm.m;          // (all loads at once: what lies past the count is not used)
    const int l0 = lst[0], l1 = lst[e1], l2 = lst[e2];
    const uint64_t i0 = cnt > 0 ? (uint32_t)l0 & 4095 : 4095, i1 = cnt > 1 ? (uint32_t)l1 & 4095 : 4095, i2 = cnt > 2 ? (uint32_t)l2 & 4095 : 4095;
    const uint64_t load = min(max(cnt, 1), dm.m) + switch_cost;                          // < 2^13
    // (every index < RSA_MAX_BLOCKS = 2^12)
    keys[i] = i < dm.n ? ((i0 << 36) | (i1 << 24) | (i2 << 12) | (uint64_t)i) << 13 | load : ~0ull;
  }
  __syncthreads();
  const int r = blockIdx.x * kRankRows + tid / 4;
  const uint64_t mine = keys[min(r, dm.n - 1)];
  int below = 0, load = 0;
  for (int i = tid % 4; i < padded; i += 32) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint64_t key = keys[i + 4 * k];
      below += key < mine ? 1 : 0;
      load += key < mine ? (int)(key & 8191) : 0;
    }
  }
  below += __shfl_xor(below, 1);
  below += __shfl_xor(below, 2);
  load += __shfl_xor(load, 1);
  load += __shfl_xor(load, 2);
  if (r < dm.n && tid % 4 == 0) a.row_order[(size_t)bh * dm.n + below] = order_entry(r, load);
}

// Minimum over the 64 lanes of a wave with data-parallel-primitive moves (row shifts inside the rows of
// 16 lanes, then the two row broadcasts): lane 63 ends up with it. Lanes without a source take INT_MAX.
__device__ __forceinline__ int wave_min_i32(int v) {
  constexpr int kMax = 0x7fffffff;
  v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x111, 0xf, 0xf, false));   // row_shr:1
  v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x112, 0xf, 0xf, false));   // row_shr:2
  v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x114, 0xf, 0xf, false));   // row_shr:4
  v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x118, 0xf, 0xf, false));   // row_shr:8
  v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x142, 0xa, 0xf, false));   // row_bcast:15 into rows 1 and 3
  v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x143, 0xc, 0xf, false));   // row_bcast:31 into rows 2 and 3
  return __builtin_amdgcn_readlane(v, 63);
}
// Sums the same way (data-parallel-primitive moves: six dependent instructions; a shuffle goes through the LDS crossbar).
__device__ __forceinline__ int wave_inclusive_scan_i32(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}
__device__ __forceinline__ int last_lane(int v) { return __builtin_amdgcn_readlane(v, 63); }
__device__ __forceinline__ int wave_sum_i32(int v) { return last_lane(wave_inclusive_scan_i32(v)); }
__device__ __forceinline__ int lanes_below(unsigned long long mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// Deals the items of one launch to the slots of the persistent attention kernel (a slot = one group of
// waves of one resident workgroup). One workgroup per queue; the slots of a queue run on one XCD. The
// queue's items: its share of the video rows, da.heads_at_once heads at a time (see heads_at_once in attn_sched.hpp),
// and its share of the text query blocks.
//
// The rows go out in rounds by one wave, a lane per slot (SPL slots per lane): in a round every slot whose load
// (key blocks so far) is within one item of the lightest takes the next item, in slot order -- neighbouring
// items go to neighbouring slots at about the same time, so that groups resident together walk similar lists.
//
// What is left at the end -- fewer rows than slots when all lists are equally long, up to twice as many
// otherwise -- and the long text rows are cut (video rows only where that is faster, see there): laid end to end and
// divided over the slots so that every slot ends at the same key block, give or take min_piece. A row that is cut is
// put together by merge_kernel. Cut points closer than min_piece to the end of a row move there. Without that, an uneven last round
// leaves slots idle (159 blocks of 24 heads on 512 slots: 7.45 rounds took 8; the dense layer of that shape
// 4.25 -> 4.08 ms) and a text row, which walks all M blocks, can be longer than the whole share of a slot
// (3 heads of 931 blocks, 6 text rows: a slot's share is 522 blocks; attention 2.79 -> 1.95 ms). In the smallest
// calls every row is its own round (2 heads of 17 blocks: 23.6 -> 11 us and 4 us of merging). Cuts need piece buffers;
// without them (pieces_per_queue 0: enough rounds that it does not matter, or no room) the long rows go first and the
// last rows one at a time to the lightest slot.
// The dealing itself takes 6-11 us up to 4000 items and 18-32 us at 22 000 to 28 000, beside the compensation that
// shares the launch (the last 128 rows one at a time took 38 us at 3816 items). It is one chain of latencies: sums over the
// slots that went through the LDS crossbar, and a search of the line for both ends of a slot's part and twice more, were a
// quarter of it (2 heads of 17 blocks: attention 20.7 -> 18.6 us).
// One queue for all slots of an XCD: with block 64 an XCD has 128 slots, and two queues of 64 on distant ranges of
// the row order shared less of its L2 (24 heads of 1182 blocks: attention 9.80 -> 9.03 ms).
constexpr int kDealSegment = 2048;   // rows of a queue staged in LDS at a time
constexpr int kTailMax = 512;        // at most kTailDense + kMaxCross + 2 kMaxSlots - 1 entries are cut
static_assert(kTailDense + kMaxCross + 2 * kMaxSlots <= kTailMax && 2 * kMaxSlots <= kDealSegment, "the tail fits its arrays and one segment");
constexpr int kDealLdsInts = 2 * kDealSegment + 3 * kTailMax + 1 + 2 * kMaxSlots + 2 * kQueues + kMaxTurns * (kQueues + 1) + 4;

template <int SPL>
__device__ __forceinline__ void deal_queue(const Dims& dm, const AttnArgs& a, const DealArgs& da, int q, uint32_t* lds) {
  constexpr int SEG = kDealSegment;
  int32_t* rec = reinterpret_cast<int32_t*>(lds);
  int32_t* len = rec + SEG;
  int32_t* t_rec = len + SEG;                     // the tail: row, first entry | (1 + cross row) << 16, start on the line
  int32_t* t_fc = t_rec + kTailMax;
  int32_t* t_pos = t_fc + kTailMax;
  int32_t* s_load = t_pos + kTailMax + 1;         // by slot
  int32_t* s_cnt = s_load + kMaxSlots;
  int32_t* s_cross = s_cnt + kMaxSlots;           // [8][2]: first and last piece of this queue's part of a cross row
  int32_t* t_cut = rec;                           // (the tail no longer needs the staged rows) pieces of an entry
  int32_t* s_part = s_cross + 2 * kQueues;        // [turns][9]: first row of every queue's part of a turn
  int32_t* s_left = s_part + kMaxTurns * (kQueues + 1);   // rows of the last segment to be dealt: from, to; equal; tail entries
  const int tid = threadIdx.x, lane = tid % 64;
  const bool dense_all = (a.flags & RSA_DENSE) != 0;
  const int bh_total = dm.batch * dm.heads, NR = da.rows_per_bh, S = da.slots;
  const bool split = da.pieces_per_queue > 0;
  const int n_whole = da.n_dense - da.n_cross;
  const int my_dense = q < n_whole ? (n_whole - q + kQueues - 1) / kQueues : 0;
  const int lead = (split && my_dense <= kTailDense) ? 0 : my_dense;         // text rows dealt whole, ahead of the others
  const int tail_dense = my_dense - lead;
  // Shares. Heads are taken da.heads_at_once at a time (a turn), their rows head by head in launch order, and cut into eight
  // parts; which part a queue gets turns. s_part[i][p]: where part p of turn i starts.
  const int at_once = da.heads_at_once, turns = (bh_total + at_once - 1) / at_once;
  const int32_t* order = dense_all ? nullptr : a.row_order;
  auto rows_of_turn = [&](int i) __attribute__((always_inline)) { return min(at_once, bh_total - i * at_once) * NR; };
  auto total_load = [&](int h) __attribute__((always_inline)) {
    return h < SEG ? len[h] : order_load(order[(size_t)h * NR + NR - 1]) + 1;
  };
  auto sum_over_turns = [&](const int32_t* at, int queue) __attribute__((always_inline)) {
    int n = 0;
    for (int i = 0; i < turns; ++i) {
      const int32_t* p = at + i * (kQueues + 1) + (queue + i) % kQueues;
      n += p[1] - p[0];
    }
    return n;
  };
  auto largest_and_sum = [&](const int32_t* at, int& sum) __attribute__((always_inline)) {      // over the queues
    if (tid < kQueues) s_cross[tid] = sum_over_turns(at, tid);
    __syncthreads();
    int most = 0;
    sum = 0;
    for (int k = 0; k < kQueues; ++k) {
      most = max(most, s_cross[k]);
      sum += s_cross[k];
    }
    __syncthreads();
    return most;
  };
  // Parts of equal numbers of rows begin and end with a head, or half or quarter of one: rows of unequal length share tiles
  // only with rows of their head. Kept as long as no queue gets over da.most_share 64ths of the average load.
  int32_t* s_total = len;                          // (nothing is staged yet) loads of the heads
  if (order)
    for (int h = tid; h < min(bh_total, SEG); h += 256) s_total[h] = order_load(order[(size_t)h * NR + NR - 1]) + 1;
  for (int k = tid; k < turns * (kQueues + 1); k += 256) {
    const int i = k / (kQueues + 1), p = k % (kQueues + 1), rows = rows_of_turn(i), at = (int)((long long)p * rows / kQueues);
    s_part[k] = at;
    if (order) rec[k] = at < rows ? order_load(order[(size_t)i * at_once * NR + at]) : 0;
  }
  __syncthreads();
  if (order) {
    for (int k = tid; k < turns * (kQueues + 1); k += 256) {
      const int i = k / (kQueues + 1), heads = s_part[k] / NR;
      for (int h = 0; h < heads; ++h) rec[k] += total_load(i * at_once + h);
    }
    __syncthreads();
  }
  bool by_load = false;
  if (order) {
    int sum;
    const int most = largest_and_sum(rec, sum);
    by_load = (long long)most * kQueues * 64 > (long long)sum * da.most_share;
  }
  if (by_load) {
    for (int k = tid; k < turns * (kQueues + 1); k += 256) {
      const int i = k / (kQueues + 1), p = k % (kQueues + 1), heads = rows_of_turn(i) / NR;
      if (p == 0 || p == kQueues) continue;
      const int32_t* o = order + (size_t)i * at_once * NR;
      int all = 0, h = 0;
      for (int j = 0; j < heads; ++j) all += total_load(i * at_once + j);
      int target = (int)((long long)p * all / kQueues);
      for (int t = 0; h + 1 < heads && target >= (t = total_load(i * at_once + h)); ++h) target -= t;
      int lo = 0, hi = NR - 1;                                   // the first row of head h that has the target before it
      while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (order_load(o[(size_t)h * NR + mid]) >= target) hi = mid;
        else lo = mid + 1;
      }
      s_part[k] = h * NR + lo;
    }
    __syncthreads();
    // A queue of very short rows might get more of them than its table holds: equal numbers of rows after all. Everything
    // that goes into the table counts, text rows that may be cut and parts of cross rows too: whatever is given out,
    // some slot then has cap - 2 entries at most (the whole entries of a line that is not cut ask for such a slot). All queues
    // have to decide alike, or their rows overlap and leave gaps: the most text rows of any queue, not this one's.
    const int most_dense = (n_whole + kQueues - 1) / kQueues;
    int sum;
    if (most_dense + da.n_cross + largest_and_sum(s_part, sum) > S * (da.cap - 2)) {
      for (int k = tid; k < turns * (kQueues + 1); k += 256)
        s_part[k] = (int)((long long)(k % (kQueues + 1)) * rows_of_turn(k / (kQueues + 1)) / kQueues);
      __syncthreads();
    }
  }
  const int n_rows = sum_over_turns(s_part, q);
  const int n_bulk = lead + n_rows;
  auto dense_record = [&](int d) __attribute__((always_inline)) {
    return (d / da.dense_per_bh) * RSA_MAX_BLOCKS + da.dense_first + d % da.dense_per_bh;
  };
  auto row_record = [&](int v) __attribute__((always_inline)) {          // v-th row of this queue
    int at = v, i = 0;
    for (; i + 1 < turns; ++i) {
      const int32_t* p = s_part + i * (kQueues + 1) + (q + i) % kQueues;
      if (at < p[1] - p[0]) break;
      at -= p[1] - p[0];
    }
    at += s_part[i * (kQueues + 1) + (q + i) % kQueues];
    const int head = i * at_once + at / NR;
    const int qb = order ? order_row(order[(size_t)head * NR + at % NR]) : at % NR;
    return head * RSA_MAX_BLOCKS + qb;
  };

  int load[SPL], cnt[SPL];
  bool ok[SPL];
#pragma unroll
  for (int j = 0; j < SPL; ++j) {
    load[j] = cnt[j] = 0;
    ok[j] = lane + 64 * j < S;
  }
  auto put = [&](int u, int at, int record, int span) __attribute__((always_inline)) {
    da.table[((size_t)q * S + u) * da.cap + at] = make_int2(record, span);
  };
  // one round over rows next .. limit-1 of the staged segment; the lightest slots only when `strict`
  auto deal_round = [&](int next, int limit, bool strict) __attribute__((always_inline)) {
    int l = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < SPL; ++j) l = min(l, ok[j] && cnt[j] < da.cap - 1 ? load[j] : 0x7fffffff);
    const int lightest = wave_min_i32(l);
    const int reach = strict ? lightest + 1 : lightest + len[next];
    bool any = false;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      const bool take = ok[j] && cnt[j] < da.cap - 1 && load[j] < reach;
      const unsigned long long takers = __ballot(take);
      const int mine = next + lanes_below(takers);
      if (take && mine < limit) {
        put(lane + 64 * j, cnt[j], rec[mine], make_span(0, len[mine], false));
        load[j] += len[mine];
        cnt[j] += 1;
      }
      any = any || takers != 0;
      next = min(limit, next + __popcll(takers));
    }
    return any ? next : limit;         // (the table has room for all rows, so some slot always takes)
  };
  // Segments of SEG rows, the odd one first, so that the tail lies in the last one.
  int seg0 = 0;
  do {
    const int left = n_bulk - seg0;
    const int seg_n = left <= 0 ? 0 : (left - 1) % SEG + 1;
    const bool last = seg0 + seg_n >= n_bulk;
    __syncthreads();
    for (int i = tid; i < seg_n; i += 256) {
      const int it = seg0 + i;
      const int r = it < lead ? dense_record(q + it * kQueues) : row_record(it - lead);
      const int qb = r % RSA_MAX_BLOCKS;
      rec[i] = r;
      len[i] = !dense_all && qb < dm.n ? list_length(a, dm, (size_t)(r / RSA_MAX_BLOCKS) * dm.n + qb) : dm.m;
    }
    __syncthreads();
    if (tid < 64) {
      int next = 0;
      const int bulk_end = seg_n - 2 * S;          // (of the last segment)
      while (next < seg_n && (!last || next <= bulk_end)) next = deal_round(next, seg_n, false);
      if (last) {
        bool equal = false, cut = split;
        if (split) {
          int lo = 0x7fffffff, hi = 0x7fffffff, flo = 0x7fffffff, fhi = 0x7fffffff;
#pragma unroll
          for (int j = 0; j < SPL; ++j)
            if (ok[j]) {
              flo = min(flo, load[j]);
              fhi = min(fhi, -load[j]);
            }
          for (int i = next + lane; i < seg_n; i += 64) {
            lo = min(lo, len[i]);
            hi = min(hi, -len[i]);
          }
          equal = wave_min_i32(flo) == -wave_min_i32(fhi) && (next >= seg_n || wave_min_i32(lo) == -wave_min_i32(hi));
          // Which video rows are cut (what is left of RSA_DENSE: as the host has decided). Text rows are cut in any case, and
          // equal rows beside them. Unequal rows are cut, but at d = 128 with blocks of 64 only when they are no more than the
          // slots and, without text rows, for half of the slots at most and not short (us, whole and cut, lists of a tenth to
          // a half of the blocks at random: 3 heads of 106 blocks, 39 rows for 128 slots 105 and 67; 24 of 13, 39 rows 33 and
          // 38; 8 of 192, 192 rows 333 and 425; 3 of 362, 136 rows 487 and 608; with two text blocks 3 of 490 1016 and 1233).
          if (!dense_all && next < seg_n) {
            if (equal) cut = da.n_dense > 0 || cut_pays(da.rule, (seg_n - next) % S, S, len[next]);
            else if (dm.d == 128 && dm.blk == 64)
              cut = n_bulk <= S && (da.n_dense > 0 || (2 * n_bulk <= S && (dm.m >= 24 || 10 * n_bulk <= S)));
          }
        }
        // whole rounds of equal rows that the rest is cut of, or all rows
        const int stop = !cut ? 1 : equal ? S : seg_n + 1;
        while (seg_n - next >= stop) next = deal_round(next, seg_n, true);
        if (split && lane == 0) {
          s_left[0] = next;
          s_left[1] = seg_n;
          s_left[2] = equal ? 1 : 0;
          s_left[3] = tail_dense + da.n_cross + seg_n - next;
        }
      }
    }
    seg0 += seg_n;
  } while (seg0 < n_bulk);

  if (!split) {
    if (tid < 64) {
#pragma unroll
      for (int j = 0; j < SPL; ++j)
        if (ok[j]) {
          const int slot = q * S + lane + 64 * j;
          da.nitems[slot] = cnt[j];
          da.total[slot] = load[j];
          da.piece0[slot] = 0;
        }
    }
    return;
  }

  // ---- the tail: text rows, this queue's parts of the cross rows, the rows left ----------------------
  if (tid < 64) {
#pragma unroll
    for (int j = 0; j < SPL; ++j)
      if (ok[j]) {
        s_load[lane + 64 * j] = load[j];
        s_cnt[lane + 64 * j] = cnt[j];
      }
    if (lane < 2 * kQueues) s_cross[lane] = lane % 2 ? -1 : 0;      // (no pieces: first 0, last -1)
  }
  __syncthreads();
  const int left0 = s_left[0], TN = s_left[3];
  const bool equal = s_left[2] != 0;
  for (int i = tid; i < TN; i += 256) {
    int r, first = 0, l, cross = 0;
    if (i < tail_dense) {
      r = dense_record(q + i * kQueues);
      l = dm.m;
    } else if (i < tail_dense + da.n_cross) {
      const int j = i - tail_dense;
      r = dense_record(n_whole + j);
      first = (int)((long long)q * dm.m / kQueues);
      l = (int)((long long)(q + 1) * dm.m / kQueues) - first;
      cross = j + 1;
    } else {
      const int k = left0 + i - tail_dense - da.n_cross;
      r = rec[k];
      l = len[k];
    }
    t_rec[i] = r;
    t_fc[i] = first | cross << 16;
    t_pos[i] = l;
  }
  __syncthreads();
  for (int i = tid; i < TN; i += 256) t_cut[i] = 0;
  __syncthreads();
  if (tid >= 64) return;                           // one wave from here on
  int line = 0;                                    // the tail laid end to end: entry i from t_pos[i] to t_pos[i + 1]
  const int len0 = TN > 0 ? t_pos[TN - 1] : 0;     // (the length of a row, when all are equal)
  for (int c = 0; c < TN; c += 64) {
    const int v = c + lane < TN ? t_pos[c + lane] : 0;
    const int incl = wave_inclusive_scan_i32(v);
    asm volatile("" ::: "memory");
    if (c + lane < TN) t_pos[c + lane] = line + incl - v;
    line += last_lane(incl);
  }
  if (lane == 0) t_pos[TN] = line;
  asm volatile("" ::: "memory");
  // Slots in the order in which they take the line: one group of every workgroup first, so that a short line
  // spreads over the CUs.
  const int W = S / da.groups;
  int u[SPL], base[SPL];
#pragma unroll
  for (int j = 0; j < SPL; ++j) {
    const int sp = lane + 64 * j;
    u[j] = ok[j] ? (sp % W) * da.groups + sp / W : 0;
    base[j] = ok[j] ? s_load[u[j]] : 0x3fffffff;
    cnt[j] = ok[j] ? s_cnt[u[j]] : 0;
  }
  // The level at which the line is used up: slots above it take nothing, and leaving them out of the average
  // lowers it, so a few steps from the average over all slots reach it from above.
  int level = 0x3ffffffe;
  for (int step = 0; step < 4; ++step) {
    int sum = 0, act = 0;
#pragma unroll
    for (int j = 0; j < SPL; ++j)
      if (base[j] < level) {
        sum += base[j];
        act += 1;
      }
    sum = wave_sum_i32(sum);
    act = wave_sum_i32(act);
    if (act == 0) break;                           // (nothing left, all loads equal)
    level = (sum + line + act - 1) / act;
  }
  int lo = 0x7fffffff;
#pragma unroll
  for (int j = 0; j < SPL; ++j) lo = min(lo, base[j]);
  lo = wave_min_i32(lo);
  level = max(level, lo + da.min_piece);
  // equal rows with nothing long among them: cutting them saves (S - rows) / S of a row and costs a switch
  if (equal && tail_dense + da.n_cross == 0 && (long long)S * len0 - line < (long long)S * da.switch_cost) level = lo + len0;
  int from[SPL], to[SPL];
  {
    int at = 0;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      const int room = max(0, level - base[j]);                  // (slots that do not exist: none)
      const int incl = wave_inclusive_scan_i32(room);
      from[j] = at + incl - room;
      to[j] = at + incl;
      at += last_lane(incl);
    }
  }
  auto entry_at = [&](int x) __attribute__((always_inline)) {     // the entry that x lies in (x < line)
    int l = 0, h = TN - 1;
    while (l < h) {
      const int mid = (l + h + 1) / 2;
      if (t_pos[mid] <= x) l = mid;
      else h = mid - 1;
    }
    return l;
  };
  struct Cut { int pos, entry; };                                 // where, and the entry that begins or goes on there
  auto cut_at = [&](int x) __attribute__((always_inline)) {
    if (x >= line) return Cut{line, TN};
    const int i = entry_at(x);
    const int p = t_pos[i], e = t_pos[i + 1], h = min(da.min_piece, (e - p + 1) / 2);
    return x - p < h ? Cut{p, i} : (e - x < h ? Cut{e, i + 1} : Cut{x, i});
  };
  // A slot takes the line from its cut to that of the next slot.
  int start[SPL];
  {
    Cut c[SPL];
#pragma unroll
    for (int j = 0; j < SPL; ++j) c[j] = cut_at(from[j]);
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      int next = __shfl_down(c[j].pos, 1);
      if (j + 1 < SPL) {
        const int first = __builtin_amdgcn_readfirstlane(c[(j + 1) % SPL].pos);
        if (lane == 63) next = first;
      } else if (lane == 63) {
        next = cut_at(to[j]).pos;
      }
      from[j] = c[j].pos;
      to[j] = next;
      start[j] = c[j].entry;
    }
  }
  int n_new[SPL], n_part[SPL], id0[SPL], pieces = 0;
  bool fits = true;
#pragma unroll
  for (int j = 0; j < SPL; ++j) {
    n_new[j] = n_part[j] = 0;
    if (ok[j]) {
      int pos = from[j];
      for (int i = start[j]; i < TN && pos < to[j]; ++i) {
        const int e = min(t_pos[i + 1], to[j]);
        if (e <= pos) continue;
        n_new[j] += 1;
        n_part[j] += (pos != t_pos[i] || e != t_pos[i + 1] || (t_fc[i] >> 16)) ? 1 : 0;
        atomicAdd(&t_cut[i], 1);                 // (LDS; a count, whatever the order)
        pos = e;
      }
      fits = fits && cnt[j] + n_new[j] <= da.cap;
    }
    const int incl = wave_inclusive_scan_i32(n_part[j]);
    id0[j] = pieces + incl - n_part[j];
    pieces += last_lane(incl);
  }
  fits = __ballot(!fits) == 0 && pieces <= da.pieces_per_queue;
  int total[SPL];
#pragma unroll
  for (int j = 0; j < SPL; ++j) total[j] = ok[j] ? base[j] : 0;
  int2* info = da.piece_info + (size_t)q * da.pieces_per_queue;
  if (fits) {
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      if (!ok[j]) continue;
      int pos = from[j], id = id0[j];
      for (int i = start[j]; i < TN && pos < to[j]; ++i) {
        const int p = t_pos[i], pe = t_pos[i + 1], e = min(pe, to[j]);
        if (e <= pos) continue;
        const int cross = t_fc[i] >> 16;
        const bool partial = pos != p || e != pe || cross;
        put(u[j], cnt[j], t_rec[i], make_span((t_fc[i] & 0xffff) + pos - p, e - pos, partial));
        cnt[j] += 1;
        total[j] += e - pos;
        if (partial) {
          info[id] = make_int2(t_rec[i], pos == p && !cross ? t_cut[i] : 0);
          if (cross && pos == p) s_cross[2 * (cross - 1)] = id;
          if (cross && e == pe) s_cross[2 * (cross - 1) + 1] = id;
          id += 1;
        }
        pos = e;
      }
    }
  } else {
    // (the table has no room for the cuts: very unequal rows) whole entries, one at a time to the lightest slot that has room:
    // there is one, shares by load leave it (see above), and by number a queue has about the average that cap is twice of
    pieces = da.n_cross;
#pragma unroll
    for (int j = 0; j < SPL; ++j) id0[j] = j == 0 && lane < da.n_cross ? lane : 0;
    for (int i = 0; i < TN; ++i) {
      const int l = t_pos[i + 1] - t_pos[i], cross = t_fc[i] >> 16;
      if (l <= 0) continue;
      int best = 0x7fffffff;
#pragma unroll
      for (int j = 0; j < SPL; ++j) best = min(best, ok[j] && cnt[j] < da.cap - 1 ? total[j] : 0x7fffffff);
      best = wave_min_i32(best);
      bool given = false;
#pragma unroll
      for (int j = 0; j < SPL; ++j) {
        // a cross part goes to the slot of its number: one piece per slot
        const unsigned long long light = __ballot(ok[j] && cnt[j] < da.cap - 1 && total[j] == best);
        const bool mine = cross ? (j == 0 && lane == cross - 1) : (!given && light && lane == __builtin_ctzll(light));
        given = given || light != 0;
        if (mine) {
          put(u[j], cnt[j], t_rec[i], make_span(t_fc[i] & 0xffff, l, cross != 0));
          cnt[j] += 1;
          total[j] += l;
          if (cross) {
            info[cross - 1] = make_int2(t_rec[i], 0);
            s_cross[2 * (cross - 1)] = s_cross[2 * (cross - 1) + 1] = cross - 1;
          }
        }
      }
    }
  }
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < SPL; ++j)
    if (ok[j]) {
      const int slot = q * S + u[j];
      da.nitems[slot] = cnt[j];
      da.total[slot] = total[j];
      da.piece0[slot] = id0[j];
    }
  for (int i = pieces + lane; i < da.pieces_per_queue; i += 64) info[i] = make_int2(-1, 0);
  if (lane < kQueues) da.cross[q * kQueues + lane] = make_int2(s_cross[2 * lane], s_cross[2 * lane + 1]);
}

__device__ __forceinline__ void deal_queue_any(const Dims& dm, const AttnArgs& a, const DealArgs& da, int q, uint32_t* lds) {
  if (da.slots <= 64) deal_queue<1>(dm, a, da, q, lds);
  else deal_queue<2>(dm, a, da, q, lds);
}
__global__ __launch_bounds__(256) void schedule_kernel(Dims dm, AttnArgs a, DealArgs da) {
  extern __shared__ uint32_t side_lds[];
  deal_queue_any(dm, a, da, blockIdx.x, side_lds);
}

// Both of the above in one launch (neither needs the other's result, and the few workgroups that deal
// the queues would otherwise have the chip to themselves): plane 0 of the grid deals queue blockIdx.x,
// plane 1 + bh compensates the rows of (batch, head) bh. The dealing workgroups are dispatched first.
template <int D>
__global__ __launch_bounds__(256) void compensation_schedule_kernel(Dims dm, AttnArgs a, DealArgs da) {
  extern __shared__ uint32_t side_lds[];
  if (blockIdx.y == 0) {
    if ((int)blockIdx.x < kQueues) deal_queue_any(dm, a, da, blockIdx.x, side_lds);   // uniform over the workgroup
    return;
  }
  if ((int)blockIdx.x * 32 < dm.n) compensate_tile<D>(dm, a, blockIdx.x * 32, (int)blockIdx.y - 1, side_lds);
}

// The rows that were cut: O = R_n * (sum over pieces of 2^(m_p - m) acc_p) / (sum of 2^(m_p - m) l_p) + C_n with
// m the largest reference of the pieces (text rows: neither R_n nor C_n), always in the order of the key blocks.
// Latency is all there is to it (a few dozen megabytes at most, out of the L2 or the Infinity Cache): one
// workgroup per piece buffer and 32 channels, of which those with the first piece of a row do its work (the
// pieces of a row are consecutive) and one per cross row and 32 channels (a run of pieces in every queue); four
// pieces are on their way at a time. A wave holds 32 query rows in the layout of 32 x 32 accumulators, a row and four
// channels to a lane, which is the order that the attention kernel writes its pieces in: read 1 KB per instruction.
template <int D, int BLK>
__global__ __launch_bounds__(64 * (BLK / 32)) void merge_kernel(Dims dm, AttnArgs a, DealArgs da) {
  constexpr int NT = 64 * (BLK / 32);
  __shared__ int32_t ids[kQueues * (2 * kMaxSlots + kMaxCross)];       // the row's piece buffers, in the order of its key blocks
  const int P = da.pieces_per_queue, dt = blockIdx.y;
  int n_run = 0;
  if ((int)blockIdx.x < kQueues * P) {
    n_run = da.piece_info[blockIdx.x].y;
    if (n_run == 0) return;                        // not the first piece of a row
    for (int i = threadIdx.x; i < n_run; i += NT) ids[i] = blockIdx.x + i;
  } else {
    const int j = (int)blockIdx.x - kQueues * P;
    int2 run[kQueues];
#pragma unroll
    for (int r = 0; r < kQueues; ++r) run[r] = da.cross[r * kQueues + j];
#pragma unroll
    for (int r = 0; r < kQueues; ++r) {
      const int n = run[r].y - run[r].x + 1;
      for (int i = threadIdx.x; i < n; i += NT) ids[n_run + i] = r * P + run[r].x + i;
      n_run += n;
    }
    if (n_run == 0) return;                        // (a cross row without pieces: cannot be)
  }
  __syncthreads();
  const int rec = da.piece_info[ids[0]].x;
  const int bh = rec / RSA_MAX_BLOCKS, qb = rec % RSA_MAX_BLOCKS;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, l32 = lane % 32, hf = lane / 32;
  const int row = wave * 32 + l32;
  const bool sparse = !(a.flags & RSA_DENSE) && qb < dm.n;
  const size_t vrow = (size_t)bh * dm.n + qb;
  const float rfac = (sparse && (a.flags & RSA_RECTIFY_CRITICAL)) ? a.R[vrow] : 1.0f;
  floatx4 c[4], acc[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    acc[g] = c[g] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (sparse && (a.flags & RSA_COMPENSATE)) c[g] = *reinterpret_cast<const floatx4*>(a.comp + vrow * D + 32 * dt + 8 * g + 4 * hf);
  }
  float m = -INFINITY, l = 0.f;
  for (int i = 0; i < n_run; i += 4) {
    float mp[4], lp[4];
    floatx4 v[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float* p = da.pieces + (size_t)ids[min(i + k, n_run - 1)] * piece_floats(D, BLK);
      lp[k] = p[BLK * D + row];
      mp[k] = i + k < n_run ? p[BLK * D + BLK + row] : -INFINITY;      // (a piece past the end: the last one, read and left out)
      const floatx4* src = reinterpret_cast<const floatx4*>(p) + (size_t)((wave * (D / 32) + dt) * 4) * 64 + lane;
#pragma unroll
      for (int g = 0; g < 4; ++g) v[k][g] = src[g * 64];
    }
    asm volatile("" ::: "memory");                 // (all four requested here, whatever is left out below)
    const float mnew = fmaxf(fmaxf(m, fmaxf(mp[0], mp[1])), fmaxf(mp[2], mp[3]));
    const float old = __builtin_amdgcn_exp2f(m - mnew);
    m = mnew;
    l *= old;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[g][e] *= old;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i + k >= n_run) break;                   // (not added with weight 0: 0 x inf is no number)
      const float w = __builtin_amdgcn_exp2f(mp[k] - mnew);
      l = fmaf(w, lp[k], l);
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[g][e] = fmaf(w, v[k][g][e], acc[g][e]);
    }
  }
  if (row >= dm.block_count(qb)) return;
  const float f = rfac / l;
  const int64_t t = dm.block_start(qb) + row;
  uint16_t* orow = a.O + (int64_t)(bh / dm.heads) * dm.sb + (int64_t)(bh % dm.heads) * dm.sh + t * dm.st + 32 * dt + 4 * hf;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = fmaf(acc[g][e], f, c[g][e]);
    uint2 w;
    w.x = pack_bf16x2(o[0], o[1]);
    w.y = pack_bf16x2(o[2], o[3]);
    *reinterpret_cast<uint2*>(orow + 8 * g) = w;
  }
  if (a.lse && hf == 0 && dt == 0) a.lse[(size_t)bh * dm.t + t] = (m + log2f(l)) * 0.6931471805599453f;
}

template <int D>
hipError_t launch_attn_side_t(const Dims& dm, const AttnArgs& a, const DealArgs& da, bool sort_rows, bool compensate, bool deal,
                              hipStream_t s) {
  const unsigned bh = (unsigned)(dm.batch * dm.heads), tiles = (unsigned)((dm.n + 31) / 32);
  const unsigned comp_lds = comp_lds_bytes<D>(), deal_lds = kDealLdsInts * 4u;
  if (sort_rows) hipLaunchKernelGGL(row_rank_kernel, dim3((dm.n + kRankRows - 1) / kRankRows, bh), dim3(256), 0, s, dm, a, da.switch_cost);
  if (deal && compensate && bh < 65535u) {
    hipLaunchKernelGGL((compensation_schedule_kernel<D>), dim3(tiles > (unsigned)kQueues ? tiles : (unsigned)kQueues, bh + 1), dim3(256),
                       comp_lds > deal_lds ? comp_lds : deal_lds, s, dm, a, da);
  } else {
    if (compensate) hipLaunchKernelGGL((compensation_kernel<D>), dim3(tiles, bh), dim3(256), comp_lds, s, dm, a);
    if (deal) hipLaunchKernelGGL(schedule_kernel, dim3(kQueues), dim3(256), deal_lds, s, dm, a, da);
  }
  return hipGetLastError();
}

template <int D, int BLK>
hipError_t launch_attn_merge_t(const Dims& dm, const AttnArgs& a, const DealArgs& da, hipStream_t s) {
  hipLaunchKernelGGL((merge_kernel<D, BLK>), dim3((unsigned)(kQueues * da.pieces_per_queue + da.n_cross), D / 32), dim3(64 * (BLK / 32)), 0, s, dm, a, da);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_side(const Dims& dm, const AttnArgs& a, const DealArgs& da, bool sort_rows, bool compensate, bool deal,
                            hipStream_t s) {
  if (dm.d == 128) return launch_attn_side_t<128>(dm, a, da, sort_rows, compensate, deal, s);
  return launch_attn_side_t<64>(dm, a, da, sort_rows, compensate, deal, s);
}

hipError_t launch_attn_merge(const Dims& dm, const AttnArgs& a, const DealArgs& da, hipStream_t s) {
  if (dm.d == 128 && dm.blk == 128) return launch_attn_merge_t<128, 128>(dm, a, da, s);
  if (dm.d == 128 && dm.blk == 64) return launch_attn_merge_t<128, 64>(dm, a, da, s);
  if (dm.d == 64 && dm.blk == 128) return launch_attn_merge_t<64, 128>(dm, a, da, s);
  return launch_attn_merge_t<64, 64>(dm, a, da, s);
}

}  // namespace rsa
