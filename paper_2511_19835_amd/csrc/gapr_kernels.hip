// Gain-Aware Pooling Rectification gate (paper Sec. 4.2; Alg. 1 steps 9-11).
//
// The relaxed condition as printed compares |sum_ij s^pool| with |sum_ij Delta s|, and the
// signed double sum of the first-order Delta s is identically zero (block means are
// subtracted). The gate therefore takes the absolute value per term, as the paper's
// un-relaxed definitions of gain and error do, on the two first-order pieces separately:
//     DA[n][m] = mean_{i in block n} |(q_i - q^pool_n) . k^pool_m| * scale
//     DB[n][m] = mean_{j in block m} |q^pool_n . (k_j - k^pool_m)| * scale
//     M_c[n][m] = |s^pool[n][m]| > DA[n][m] + DB[n][m]
// (gain and error both divided by c_n c_m). Each deviation is a skinny GEMM of a token
// block against all pooled vectors of the other side, so the cost is tokens x blocks x d.
//
// deviation_kernel: one workgroup per token block. The block is read once (on the key side the
// launch pools it as well: the only pass over K of the whole preparation), centred on its
// pooled vector (x_i - x^pool, fp32 subtraction, rounded to fp16) and parked in LDS; every
// wave then walks the pooled vectors of the other side 32 at a time against the whole centred
// block (the MFMA A operand, read from LDS half a k-step ahead), so the accumulators hold
// the deviations themselves and the epilogue is one |.|-add per element. Four waves per SIMD.
// The key side runs first and leaves DB transposed ([M][N]) in the workspace; the query side runs second
// and never stores DA: it decides the bits of M_c from its registers, S[n][m] and DBt[m][n]. Many long rows take
// deviation_long_kernel instead (below). What bounds it is the latency of its operands beside matrix work at the clock
// that power leaves: products of 16 x 16 x 32 (less power than 32 x 32 x 16), and one register set for the pooled operand, reloaded
// as it is used up, so that four waves fit a SIMD (two sets, a whole iteration ahead, three waves: 219 and 225 us where
// one takes 208 and 211). Against products of 32 x 32 x 16 with two sets, key side and query side, us, medians of three runs of either in
// turn: 24 heads of 516 blocks 226 -> 216 and 235 -> 219, 24 of 159 46 -> 43 and 40 -> 39, d = 64 23.0 -> 21.5 and
// 19.7 -> 18.2; blocks of 64, 24 of 317 76 -> 69 and 77 -> 76, 24 of 512 157 -> 141 and 167 -> 165, 1 of 1182 32 -> 28 and
// 33 -> 31. The pooled operand is rounded to fp16 as well; accumulation is fp32. fp16 rather than bf16 because both operands are O(1)
// quantities whose 2^-12 relative rounding leaves DA / DB within 2e-4 relative of fp64
// arithmetic (bf16 operands: up to 1.5e-3, wider than the 1e-3 band in which the gate may
// differ); the MFMA rate is the same. Conversions saturate at the largest finite half.
#include <type_traits>

#include "rsa_common.hpp"
#include "text_mass.hpp"

namespace rsa {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#ifndef RSA_DEV_NT
#define RSA_DEV_NT 256
#endif

// 16-byte chunk c of row r sits at chunk position c ^ key(r): 16 consecutive rows read at one
// logical chunk index then touch every LDS bank once. CPR = chunks per row (8 or 16).
template <int CPR>
__device__ __forceinline__ int swizzled(int r, int c) { return r * CPR + (c ^ ((r / (16 / CPR)) & (CPR - 1))); }

#ifndef RSA_DEV_OCC
#define RSA_DEV_OCC 4
#endif
// The first workgroups of a key-side launch, `text_wgs` for every (batch, head), make the text log-masses (they need
// the pooled queries, like this launch, and the implicit attention that follows needs them). Counts them off `wg`.
template <int D, int BLK>
__device__ __forceinline__ bool text_block(const Dims& dm, const ScoreArgs& text, int text_wgs, int& wg, float* lds) {
  const int all = text_wgs * dm.batch * dm.heads;
  if (wg < all) {
    text_mass_block<D, BLK>(dm, text, wg % text_wgs, wg / text_wgs, lds);
    return true;
  }
  wg -= all;
  return false;
}

// GATE: the launch for the query side, run second. Its deviations DA[n][.] never leave the registers:
// with the pooled score S[n][m] and the key-side deviation DBt[m][n] of the first launch (one word each
// per lane and iteration, asked for at the start of the iteration) the lane decides its bit of M_c, and
// a ballot makes the mask word of the iteration.
// The key side also makes the pooled vector of its block -- it holds the whole block in
// registers before it centres it -- and writes it (fp32, and the fp16 operand copy) for the kernels that
// follow, with the arithmetic of pool_qk_kernel (same thread-to-row mapping, same order of additions), so
// the separate pooling pass over K is not needed.
template <int D, int BLK, int NT, bool GATE>
__global__ __launch_bounds__(NT, RSA_DEV_OCC) void deviation_kernel(Dims dm, const uint16_t* __restrict__ X,
                                                           const float* __restrict__ Xpool, float* __restrict__ Xpool_out,
                                                           uint16_t* __restrict__ Xpool_f16_out, int n_blocks_x,
                                                           const uint16_t* __restrict__ PB,
                                                           int n_other, float* __restrict__ out,
                                                           const float* __restrict__ Spool,
                                                           const float* __restrict__ DBt,
                                                           uint32_t* __restrict__ Mc_bits, ScoreArgs text, int text_wgs) {
  constexpr int MT = BLK / 16, KS = D / 32, CPR = D / 8;   // row tiles of 16, k-steps of 32 channels
  constexpr int NW = NT / 64;                    // waves per workgroup
  constexpr int RPP = NT / CPR;                  // rows staged per pass of the workgroup
  __shared__ u32x4 atile[BLK * CPR];
  // Workgroup i runs on XCD i % 8. Each XCD takes a contiguous eighth of the (batch, head, block)
  // range, so that token blocks that are neighbours run on the same XCD at about the same time: the
  // query side reads DBt[m][n] for a fixed n, 32 neighbouring n to a 128-byte line, which then
  // comes into one L2 once instead of into all eight.
  const int total = n_blocks_x * dm.batch * dm.heads;
  int wg = blockIdx.x;
  if constexpr (!GATE) {
    if (text_block<D, BLK>(dm, text, text_wgs, wg, reinterpret_cast<float*>(atile))) return;
  }
  const int xcd = wg % 8, q8 = total / 8, r8 = total % 8;
  const int item = xcd * q8 + (xcd < r8 ? xcd : r8) + wg / 8;
  const int xb = item % n_blocks_x, bh = item / n_blocks_x;
  const int b = bh / dm.heads, h = bh % dm.heads;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int l16 = lane % 16, q = lane / 16;
  const int count = dm.block_count(xb);
  const int64_t t0 = dm.block_start(xb);
  const uint16_t* Xb = X + (int64_t)b * dm.sb + (int64_t)h * dm.sh;

  // ---- stage the centred block: thread -> chunk column tid % CPR, rows tid / CPR + RPP*i ----
  {
    const int cc = threadIdx.x % CPR, r0 = threadIdx.x / CPR;
    u32x4 raw[BLK / RPP];
#pragma unroll
    for (int i = 0; i < BLK / RPP; ++i) {
      const int r = r0 + RPP * i;
      const int rr = r < count ? r : count - 1;                  // stay inside the tensor; zeroed below
      raw[i] = *reinterpret_cast<const u32x4*>(Xb + (t0 + rr) * dm.st + 8 * cc);
    }
    floatx4 m0, m1;
    if constexpr (!GATE) {
      static_assert(NT == 256 && RPP * D * 4 <= BLK * CPR * 16, "the mapping of pool_qk_kernel; its partial sums fit the tile");
      __shared__ __align__(16) float mean_lds[D];
      float (*red)[D] = reinterpret_cast<float (*)[D]>(atile);   // the tile is written after the sums have been read
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < BLK / RPP; ++i) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (r0 + RPP * i < count) v = make_uint4(raw[i].x, raw[i].y, raw[i].z, raw[i].w);
        accumulate8(acc, v);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) red[r0][cc * 8 + e] = acc[e];
      __syncthreads();
      if (threadIdx.x < D) {
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < RPP; ++r) sum += red[r][threadIdx.x];
        const float mean = sum / (float)count;
        mean_lds[threadIdx.x] = mean;
        Xpool_out[((size_t)bh * n_blocks_x + xb) * D + threadIdx.x] = mean;
        Xpool_f16_out[(size_t)bh * gate_operand_vectors(n_blocks_x) * D + gate_operand_offset<D>(xb, threadIdx.x)] = to_f16_bits_sat(mean);
      }
      __syncthreads();
      m0 = *reinterpret_cast<const floatx4*>(mean_lds + 8 * cc);
      m1 = *reinterpret_cast<const floatx4*>(mean_lds + 8 * cc + 4);
      __syncthreads();                                             // every read of the sums is done
    } else {
      const float* mp = Xpool + ((size_t)bh * n_blocks_x + xb) * D + 8 * cc;
      m0 = *reinterpret_cast<const floatx4*>(mp);
      m1 = *reinterpret_cast<const floatx4*>(mp + 4);
    }
#pragma unroll
    for (int i = 0; i < BLK / RPP; ++i) {
      const int r = r0 + RPP * i;
      u32x4 c;
      c.x = pack_f16x2_sat(bf16_bits_to_float(raw[i].x & 0xffffu) - m0[0], bf16_bits_to_float(raw[i].x >> 16) - m0[1]);
      c.y = pack_f16x2_sat(bf16_bits_to_float(raw[i].y & 0xffffu) - m0[2], bf16_bits_to_float(raw[i].y >> 16) - m0[3]);
      c.z = pack_f16x2_sat(bf16_bits_to_float(raw[i].z & 0xffffu) - m1[0], bf16_bits_to_float(raw[i].z >> 16) - m1[1]);
      c.w = pack_f16x2_sat(bf16_bits_to_float(raw[i].w & 0xffffu) - m1[2], bf16_bits_to_float(raw[i].w >> 16) - m1[3]);
      if (r >= count) c = u32x4{0u, 0u, 0u, 0u};                // rows past a ragged block contribute nothing
      atile[swizzled<CPR>(r, cc)] = c;
    }
  }
  __syncthreads();
  const u32x4* arow = atile + l16 * CPR;
  const int akey = (l16 / (16 / CPR)) & (CPR - 1);     // (the same for every row tile: 16 rows are whole periods of the key)

  const float outscale = dm.scale / (float)count;
  float* orow = out + ((size_t)bh * n_blocks_x + xb) * n_other;
  // pooled vectors of the other side, fp16, in the layout of gate_operand_offset: eight channels
  // of the 32 vectors of one iteration are 512 bytes in a row, 16 bytes per lane
  const uint16_t* PBh = PB + (size_t)bh * gate_operand_vectors(n_other) * D + 256 * q + 8 * l16;

  // The B operand of one iteration is 32 pooled vectors, two column tiles of 16: lane (l16, q) supplies
  // channels 32s + 8q .. +7 of vectors o0 + l16 and o0 + 16 + l16 for k-step s. Its registers are
  // reloaded for the next iteration as soon as their last product is issued. The block's row tiles are taken
  // four at a time (a pass), so only 32 accumulator registers are live. Vectors past the end of the last group
  // are padding: they only feed output columns that are never stored.
  constexpr int TP = 4;
  u32x4 bv[KS][2];
  auto load_vectors = [&](int s, int o0) __attribute__((always_inline)) {
    const uint16_t* p = PBh + (size_t)(o0 / 32) * KS * 1024 + 1024 * s;
#pragma unroll
    for (int c = 0; c < 2; ++c) bv[s][c] = *reinterpret_cast<const u32x4*>(p + 128 * c);
  };
  // The A operand (rows) is read from LDS half a k-step ahead: two of the four row tiles of a pass.
  u32x4 av[2][2];
  auto load_a = [&](int set, int half_step) __attribute__((always_inline)) {   // half_step: (pass * KS + k-step) * 2 + half
    const int s = half_step / 2 % KS, tile = half_step / 2 / KS * TP + half_step % 2 * 2;
    const u32x4* p = arow + ((4 * s + q) ^ akey) + tile * (16 * CPR);
#pragma unroll
    for (int t = 0; t < 2; ++t) av[set][t] = p[t * 16 * CPR];
  };
  auto iteration = [&](int o0, auto morec) __attribute__((always_inline)) {
    constexpr bool more = decltype(morec)::value != 0;
    const int j = o0 + lane % 32;       // the column that this lane decides or stores
    float s_val = 0.f, db_val = 0.f;
    if constexpr (GATE) {
      const int m = j < n_other ? j : n_other - 1;
      s_val = Spool[((size_t)bh * n_blocks_x + xb) * n_other + m];
      db_val = DBt[((size_t)bh * n_other + m) * n_blocks_x + xb];
    }
    // every accumulator of a lane belongs to column l16 of its tile; the rows are spread over the
    // registers, the row tiles and the four quarters of the wave
    float dv[2][2] = {{0.f, 0.f}, {0.f, 0.f}};     // two partial sums per column tile: no long chain of dependent adds
#pragma unroll
    for (int t0 = 0; t0 < MT; t0 += TP) {
      floatx4 acc[TP][2];
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int hs = (t0 / TP * KS + s) * 2 + half;
          asm volatile("" ::: "memory");      // the A operand is re-read every iteration: no hoisting into registers
          load_a((hs + 1) % 2, (hs + 1) % (MT / TP * KS * 2));
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              floatx4 c0 = acc[2 * half + t][c];
              if (s == 0) c0 = floatx4{0.f, 0.f, 0.f, 0.f};
              acc[2 * half + t][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, av[hs % 2][t]),
                                                                            __builtin_bit_cast(halfx8, bv[s][c]), c0, 0, 0, 0);
            }
          if constexpr (more) {
            if (t0 + TP == MT && half == 1) load_vectors(s, o0 + 32 * NW);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
      for (int t = 0; t < TP; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) dv[c][r % 2] += fabsf(acc[t][c][r]);
    }
    // odd quarters finish the second column tile, even ones the first: lane l holds column l % 32
    const float d0 = dv[0][0] + dv[0][1], d1 = dv[1][0] + dv[1][1];
    float d = (q & 1 ? d1 : d0) + __shfl_xor(q & 1 ? d0 : d1, 16);
    d += __shfl_xor(d, 32);
    if constexpr (GATE) {
      const bool pred = j < n_other && fabsf(s_val) > d * outscale + db_val;
      const unsigned long long word = __ballot(pred);
      if (lane == 0) Mc_bits[((size_t)bh * n_blocks_x + xb) * dm.w + o0 / 32] = (uint32_t)word;
    } else {
      if (lane < 32 && j < n_other) orow[j] = d * outscale;
    }
  };
  int o0 = 32 * wave;
  if (o0 < n_other) {
#pragma unroll
    for (int s = 0; s < KS; ++s) load_vectors(s, o0);
    load_a(0, 0);
    for (; o0 + 32 * NW < n_other; o0 += 32 * NW) iteration(o0, std::integral_constant<int, 1>{});
    iteration(o0, std::integral_constant<int, 0>{});
  }
}

constexpr int kDevRows = 128;                    // token rows of a workgroup: one block of 128 or two of 64
constexpr int kDevThreads = 256;
constexpr int kDevWaves = kDevThreads / 64;
constexpr int kDevCols = 32 * kDevWaves;         // pooled vectors of an iteration: 32 per wave

// The same two launches for long rows (use_long_rows below). What bounds the gate is its matrix work (fp16, at the clock the power
// limit leaves), so less of it is done: DA is >= 0 and rounding is monotone, so a pair with |S| <= DB has its bit
// clear whatever DA is. The query side (GATE) lists the key blocks with |S| > DB first (44 to 63 % of them on smooth
// clips) and multiplies those only, gathering their vectors out of the operand layout; the bits are the same. For
// that the key side leaves DB as [N][M], rows that the query side reads whole, ahead of its product. A workgroup
// takes 128 token rows (two blocks of 64: half the operand traffic per row, one list for both), 64 of them at a
// time and one register set for the other operand, reloaded as it is used up: four waves per SIMD on the key side,
// three on the query side. The products are of 16 x 16 x 32: those of 32 x 32 x 16 draw more power for the same work, and
// the clock is what power leaves. Key side and query side, us, products of 32 and of 16: 24 heads of 931 blocks 678 -> 590
// and 495 -> 466, 24 of 1182 blocks of 64 578 -> 500 and 543 -> 498.
// Both launches together, against the pair of launches above (us; both with products of 32 x 32 x 16): 24 heads of 931 blocks 1256 -> 1129, 40 heads of
// 591 916 -> 836, 24 heads of 1182 blocks of 64 1306 -> 1093, 3 heads of 931 174 -> 158. Building the list costs a
// workgroup about 3 us, which short rows do not earn back (24 heads of 516 blocks 437 -> 466, 2 of 17 7.2 -> 10.0) and
// a single round of workgroups cannot hide (3 heads of 636 blocks of 64: no gain): hence the two conditions.
// At d = 64, the whole of rsa_pool: 24 of 931 1030 -> 901, 40 of 591 795 -> 718, 24 of 734 blocks of 64 504 -> 397. How much is
// skipped depends on the inputs: with every pair open (blocks of equal tokens) rsa_pool takes 1753 -> 1810 us at 24 of 931 blocks of
// 128, d = 128, and 796 -> 809 at 24 of 556, no more than before at d = 64 or with blocks of 64 (1731 -> 1557 at 24 of 1182); with
// none open 1799 -> 1323.
inline bool use_long_rows(const Dims& dm) {
  const int groups = (dm.n + kDevRows / dm.blk - 1) / (kDevRows / dm.blk);
  return dm.m > 544 && (long long)groups * dm.batch * dm.heads > 1024;
}
// On the key side the launch also makes the pooled vector of its block, as in deviation_kernel.
template <int D, int BLK, bool GATE>
__global__ __launch_bounds__(kDevThreads, GATE ? 3 : 4) void deviation_long_kernel(Dims dm, const uint16_t* __restrict__ X,
                                                          const float* __restrict__ Xpool, float* __restrict__ Xpool_out,
                                                          uint16_t* __restrict__ Xpool_f16_out, int n_blocks_x,
                                                          const uint16_t* __restrict__ PB,
                                                          int n_other, float* __restrict__ out,
                                                          const float* __restrict__ Spool,
                                                          const float* __restrict__ DB,
                                                          uint32_t* __restrict__ Mc_bits, ScoreArgs text, int text_wgs) {
  constexpr int NT = kDevThreads, NW = kDevWaves;
  constexpr int KS = D / 32, CPR = D / 8;        // k-steps of 32 channels
  constexpr int RB = kDevRows / BLK;             // token blocks of the workgroup
  constexpr int NPASS = kDevRows / 64;           // passes over the k-steps, of four row tiles each
  constexpr int PB_ROWS = BLK / 64;              // passes of a token block
  constexpr int RPP = NT / CPR;                  // rows staged per pass of the workgroup
  constexpr int NP = kDevRows / RPP, PB_ = BLK / RPP;   // passes in all and of one token block
  constexpr int LU = 4 / RB;                     // chunks of 64 key blocks whose scores and deviations a wave asks for at a time
  __shared__ u32x4 atile[kDevRows * CPR];
  // Workgroup i runs on XCD i % 8. Each XCD takes a contiguous eighth of the (batch, head, block) range: the key side
  // stores DB[n][m] word by word, 32 neighbouring m to a 128-byte line, which then comes together in one L2, and the
  // pooled vectors that an XCD reads at any time are those of a head or two.
  const int groups_x = (n_blocks_x + RB - 1) / RB;
  const int total = groups_x * dm.batch * dm.heads;
  int wg = blockIdx.x;
  if constexpr (!GATE) {
    if (text_block<D, BLK>(dm, text, text_wgs, wg, reinterpret_cast<float*>(atile))) return;
  }
  const int xcd = wg % 8, q8 = total / 8, r8 = total % 8;
  const int item = xcd * q8 + (xcd < r8 ? xcd : r8) + wg / 8;
  const int xb0 = (item % groups_x) * RB, bh = item / groups_x;
  const int b = bh / dm.heads, h = bh % dm.heads;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int l16 = lane % 16, q = lane / 16;
  const uint16_t* Xb = X + (int64_t)b * dm.sb + (int64_t)h * dm.sh;
  int count[RB];                                 // rows of each token block (0: the block does not exist)
#pragma unroll
  for (int k = 0; k < RB; ++k) count[k] = xb0 + k < n_blocks_x ? dm.block_count(xb0 + k) : 0;

  // Pooled vectors of the other side: fp16, in the layout of gate_operand_offset: of 32 consecutive vectors
  // eight channels are 512 bytes in a row, those of 16 vectors two whole lines
  const uint16_t* PBh = PB + (size_t)bh * gate_operand_vectors(n_other) * D + 256 * q;

  // ---- stage the centred block: thread -> chunk column tid % CPR, rows tid / CPR + RPP*i ----
  const int cc = threadIdx.x % CPR, r0 = threadIdx.x / CPR;
  u32x4 raw[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int k = i / PB_, r = r0 + RPP * (i % PB_);
    const int xb = count[k] > 0 ? xb0 + k : xb0, cnt = count[k] > 0 ? count[k] : count[0];
    const int rr = r < cnt ? r : cnt - 1;                        // stay inside the tensor; zeroed below
    raw[i] = *reinterpret_cast<const u32x4*>(Xb + (dm.block_start(xb) + rr) * dm.st + 8 * cc);
  }
  // ---- query side: the key blocks whose bit is still open, each wave from a range of its own --------
  constexpr int LM = GATE ? RSA_MAX_BLOCKS : 1;
  __shared__ uint16_t list[LM];                                  // wave w's from w * range on
  __shared__ uint32_t words[RB][LM / 32 + 1];                    // the mask words of the token blocks
  __shared__ int list_n[NW];
  const int range = (n_other + 64 * NW - 1) / (64 * NW) * 64;       // key blocks a wave looks at
  const float* Srow = Spool + ((size_t)bh * n_blocks_x + xb0) * n_other;       // (of the first token block, like DBcol)
  const float* DBrow = DB + ((size_t)bh * n_blocks_x + xb0) * n_other;
  if constexpr (GATE) {
    for (int i = threadIdx.x; i < RB * (LM / 32 + 1); i += NT) (&words[0][0])[i] = 0u;
    const int base = wave * range;
    int n = 0;
    for (int c0 = 0; c0 < range; c0 += 64 * LU) {
      float s[LU][RB], db[LU][RB];
#pragma unroll
      for (int u = 0; u < LU; ++u) {
        const int m = base + c0 + 64 * u + lane, mm = m < n_other ? m : n_other - 1;
#pragma unroll
        for (int k = 0; k < RB; ++k) {
          const int kk = count[k] > 0 ? k : 0;
          s[u][k] = fabsf(Srow[(size_t)kk * n_other + mm]);
          db[u][k] = DBrow[(size_t)kk * n_other + mm];
        }
      }
#pragma unroll
      for (int u = 0; u < LU; ++u) {
        const int c = c0 + 64 * u + lane, m = base + c;
        bool open = false;
#pragma unroll
        for (int k = 0; k < RB; ++k) open = open || s[u][k] > db[u][k];
        open = open && c < range && m < n_other;
        const unsigned long long set = __ballot(open);
        if (open) list[base + n + __builtin_amdgcn_mbcnt_hi((uint32_t)(set >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)set, 0u))] = (uint16_t)m;
        n += __popcll(set);
      }
    }
    if (lane == 0) list_n[wave] = n;
  }
  {
    floatx4 m0[RB], m1[RB];
    if constexpr (!GATE) {
      static_assert(RB * RPP * D * 4 <= kDevRows * CPR * 16 && RB * D <= NT, "the partial sums fit the tile");
      __shared__ __align__(16) float mean_lds[RB][D];
      float (*red)[RPP][D] = reinterpret_cast<float (*)[RPP][D]>(atile);   // the tile is written after the sums have been read
#pragma unroll
      for (int k = 0; k < RB; ++k) {
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < PB_; ++i) {
          const u32x4 x = raw[k * PB_ + i];
          uint4 v = make_uint4(0, 0, 0, 0);
          if (r0 + RPP * i < count[k]) v = make_uint4(x.x, x.y, x.z, x.w);
          accumulate8(acc, v);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) red[k][r0][cc * 8 + e] = acc[e];
      }
      __syncthreads();
      if (threadIdx.x < RB * D) {
        const int k = threadIdx.x / D, c = threadIdx.x % D;
        const int cnt = k == 0 ? count[0] : count[RB - 1];
        if (cnt > 0) {
          float sum = 0.f;
#pragma unroll
          for (int r = 0; r < RPP; ++r) sum += red[k][r][c];
          const float mean = sum / (float)cnt;
          mean_lds[k][c] = mean;
          Xpool_out[((size_t)bh * n_blocks_x + xb0 + k) * D + c] = mean;
          Xpool_f16_out[(size_t)bh * gate_operand_vectors(n_blocks_x) * D + gate_operand_offset<D>(xb0 + k, c)] = to_f16_bits_sat(mean);
        } else {
          mean_lds[k][c] = 0.f;
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < RB; ++k) {
        m0[k] = *reinterpret_cast<const floatx4*>(&mean_lds[k][8 * cc]);
        m1[k] = *reinterpret_cast<const floatx4*>(&mean_lds[k][8 * cc + 4]);
      }
      __syncthreads();                                             // every read of the sums is done
    } else {
#pragma unroll
      for (int k = 0; k < RB; ++k) {
        const float* mp = Xpool + ((size_t)bh * n_blocks_x + (count[k] > 0 ? xb0 + k : xb0)) * D + 8 * cc;
        m0[k] = *reinterpret_cast<const floatx4*>(mp);
        m1[k] = *reinterpret_cast<const floatx4*>(mp + 4);
      }
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int k = i / PB_, r = r0 + RPP * (i % PB_);
      u32x4 c;
      c.x = pack_f16x2_sat(bf16_bits_to_float(raw[i].x & 0xffffu) - m0[k][0], bf16_bits_to_float(raw[i].x >> 16) - m0[k][1]);
      c.y = pack_f16x2_sat(bf16_bits_to_float(raw[i].y & 0xffffu) - m0[k][2], bf16_bits_to_float(raw[i].y >> 16) - m0[k][3]);
      c.z = pack_f16x2_sat(bf16_bits_to_float(raw[i].z & 0xffffu) - m1[k][0], bf16_bits_to_float(raw[i].z >> 16) - m1[k][1]);
      c.w = pack_f16x2_sat(bf16_bits_to_float(raw[i].w & 0xffffu) - m1[k][2], bf16_bits_to_float(raw[i].w >> 16) - m1[k][3]);
      if (r >= count[k]) c = u32x4{0u, 0u, 0u, 0u};              // rows past a ragged block contribute nothing
      atile[swizzled<CPR>(k * BLK + r, cc)] = c;
    }
  }
  __syncthreads();
  const u32x4* arow = atile + l16 * CPR;
  const int akey = (l16 / (16 / CPR)) & (CPR - 1);     // (the same for every row tile: 16 rows are whole periods of the key)

  float outscale[RB];
#pragma unroll
  for (int k = 0; k < RB; ++k) outscale[k] = dm.scale / (float)count[k];
  int n_cols = n_other, seg1 = 0, seg2 = 0, seg3 = 0;   // columns, and where the lists of waves 1 .. 3 start among them
  if constexpr (GATE) {
    seg1 = __builtin_amdgcn_readfirstlane(list_n[0]);
    seg2 = seg1 + __builtin_amdgcn_readfirstlane(list_n[1]);
    seg3 = seg2 + __builtin_amdgcn_readfirstlane(list_n[2]);
    n_cols = seg3 + __builtin_amdgcn_readfirstlane(list_n[3]);
  }
  auto block_of = [&](int j) __attribute__((always_inline)) {        // pooled vector of column j
    j = j < n_cols ? j : n_cols - 1;               // (columns past the end repeat the last one; their results are not used)
    if (!GATE) return j;
    return (int)list[j < seg1 ? j : j < seg2 ? j - seg1 + range : j < seg3 ? j - seg2 + 2 * range : j - seg3 + 3 * range];
  };
  // The B operands of an iteration are two column tiles of 16: lane (l16, q) supplies channels 32s + 8q .. +7 of columns
  // o0 + l16 and o0 + 16 + l16 in k-step s.
  const uint16_t* pv[2];
  auto find_vectors = [&](int o0) __attribute__((always_inline)) {
    if constexpr (GATE) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int m = block_of(o0 + 16 * c + l16);
        pv[c] = PBh + (size_t)(m / 32) * (KS * 1024) + (m % 32) * 8;
      }
    } else {                                       // (vectors past the end of the last 32 are padding: they feed columns that are not stored)
      pv[0] = PBh + (size_t)(o0 / 32) * (KS * 1024) + l16 * 8;
      pv[1] = pv[0] + 16 * 8;
    }
  };
  u32x4 bv[KS][2];
  u32x4 av[2][2];
  auto load_vectors = [&](int s) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 2; ++c) bv[s][c] = *reinterpret_cast<const u32x4*>(pv[c] + 1024 * s);
  };
  // half steps: two of the four row tiles of a pass
  auto load_a = [&](int set, int half_step) __attribute__((always_inline)) {   // half_step: (pass * KS + k-step) * 2 + half
    const int s = half_step / 2 % KS, tile = half_step / 2 / KS * 4 + half_step % 2 * 2;
    const u32x4* p = arow + ((4 * s + q) ^ akey) + tile * (16 * CPR);
#pragma unroll
    for (int t = 0; t < 2; ++t) av[set][t] = p[t * 16 * CPR];
  };
  // 32 columns of the wave against the 128 rows, 64 rows at a time. The A operand (rows) is read from LDS half a k-step
  // ahead; the registers of B are reloaded for the next iteration as soon as their last product is issued.
  auto iteration = [&](int o0, auto morec) __attribute__((always_inline)) {
    constexpr bool more = decltype(morec)::value != 0;
    if constexpr (more) find_vectors(o0 + kDevCols);
    const int j = o0 + lane % 32;                  // the column that this lane decides or stores
    int m = 0;
    float s_val[RB], db_val[RB];
    if constexpr (GATE) {
      m = block_of(j);
#pragma unroll
      for (int k = 0; k < RB; ++k) {
        const int kk = count[k] > 0 ? k : 0;
        s_val[k] = Srow[(size_t)kk * n_other + m];
        db_val[k] = DBrow[(size_t)kk * n_other + m];
      }
    }
    float dv[2][2];                                // two partial sums per column tile: no long chain of dependent adds
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
      floatx4 acc[4][2];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int hs = (pass * KS + s) * 2 + half;
          asm volatile("" ::: "memory");      // the A operand is re-read every iteration: no hoisting into registers
          load_a((hs + 1) % 2, (hs + 1) % (NPASS * KS * 2));
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              floatx4 c0 = acc[2 * half + t][c];
              if (s == 0) c0 = floatx4{0.f, 0.f, 0.f, 0.f};
              acc[2 * half + t][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, av[hs % 2][t]),
                                                                            __builtin_bit_cast(halfx8, bv[s][c]), c0, 0, 0, 0);
            }
          if constexpr (more) {
            if (pass == NPASS - 1 && half == 1) load_vectors(s);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // every accumulator of a lane belongs to column l16 of its tile; the rows are spread over the registers, the row
      // tiles of the block and the four quarters of the wave
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            dv[c][r % 2] = (pass % PB_ROWS == 0 && t == 0 && r < 2 ? 0.f : dv[c][r % 2]) + fabsf(acc[t][c][r]);
      if (pass % PB_ROWS == PB_ROWS - 1) {
        const int k = pass / PB_ROWS;
        // odd quarters finish the second column tile, even ones the first: lanes 0 to 31 hold the 32 columns
        const float d0 = dv[0][0] + dv[0][1], d1 = dv[1][0] + dv[1][1];
        float d = (q & 1 ? d1 : d0) + __shfl_xor(q & 1 ? d0 : d1, 16);
        d += __shfl_xor(d, 32);
        if constexpr (GATE) {
          if (lane < 32 && j < n_cols && fabsf(s_val[k]) > d * outscale[k] + db_val[k]) atomicOr(&words[k][m / 32], 1u << (m % 32));
        } else {
          // transposed, [N][M]: the query side reads whole rows. The stores are 4 bytes each, but the key blocks of
          // a line are neighbours and meet in the L2 of their XCD.
          if (lane < 32 && j < n_cols && count[k] > 0) out[((size_t)bh * n_other + j) * n_blocks_x + xb0 + k] = d * outscale[k];
        }
      }
    }
  };
  int o0 = 32 * wave;
  if (o0 < n_cols) {
    find_vectors(o0);
#pragma unroll
    for (int s = 0; s < KS; ++s) load_vectors(s);
    load_a(0, 0);
    for (; o0 + kDevCols < n_cols; o0 += kDevCols) iteration(o0, std::integral_constant<int, 1>{});
    iteration(o0, std::integral_constant<int, 0>{});
  }
  if constexpr (GATE) {
    __syncthreads();
    for (int i = threadIdx.x; i < RB * dm.w; i += NT) {
      const int k = i / dm.w, w = i % dm.w;
      if (xb0 + k < n_blocks_x) Mc_bits[((size_t)bh * n_blocks_x + xb0 + k) * dm.w + w] = words[k][w];
    }
  }
}

__global__ void fill_bits_kernel(Dims dm, uint32_t* bits, uint32_t value) {
  const size_t total = (size_t)dm.batch * dm.heads * dm.n * dm.w;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int wd = (int)(i % dm.w);
    uint32_t v = value;
    const int valid = dm.m - wd * 32;
    if (valid < 32) v &= (valid <= 0) ? 0u : ((1u << valid) - 1u);
    bits[i] = v;
  }
}

template <int D, int BLK>
hipError_t launch_gapr_keys_t(const Dims& dm, const GaprArgs& a, hipStream_t s) {
  const unsigned bh = (unsigned)(dm.batch * dm.heads);
  constexpr unsigned NT = RSA_DEV_NT, RB = kDevRows / BLK;
  ScoreArgs text = {};
  text.K = a.K; text.Qp = a.Qp; text.Lmass = a.text_Lmass;
  const int text_wgs = a.text_Lmass ? text_mass_workgroups(dm) : 0;
  if (use_long_rows(dm))
    hipLaunchKernelGGL((deviation_long_kernel<D, BLK, false>), dim3(((dm.m + RB - 1) / RB + text_wgs) * bh), dim3(kDevThreads), 0, s, dm,
                       a.K, nullptr, a.Kp_out, a.Kpb_out, dm.m, a.Qpb, dm.n, a.DB, nullptr, nullptr, nullptr, text, text_wgs);
  else
    hipLaunchKernelGGL((deviation_kernel<D, BLK, NT, false>), dim3((dm.m + text_wgs) * bh), dim3(NT), 0, s, dm, a.K, nullptr, a.Kp_out,
                       a.Kpb_out, dm.m, a.Qpb, dm.n, a.DB, nullptr, nullptr, nullptr, text, text_wgs);
  return hipGetLastError();
}
// turns its deviations into the bits of M_c on the spot
template <int D, int BLK>
hipError_t launch_gapr_queries_t(const Dims& dm, const GaprArgs& a, hipStream_t s) {
  const unsigned bh = (unsigned)(dm.batch * dm.heads);
  constexpr unsigned NT = RSA_DEV_NT, RB = kDevRows / BLK;
  if (use_long_rows(dm))
    hipLaunchKernelGGL((deviation_long_kernel<D, BLK, true>), dim3((dm.n + RB - 1) / RB * bh), dim3(kDevThreads), 0, s, dm, a.Q, a.Qp,
                       nullptr, nullptr, dm.n, a.Kpb, dm.m, nullptr, a.Spool, a.DB, a.Mc_bits, ScoreArgs{}, 0);
  else
    hipLaunchKernelGGL((deviation_kernel<D, BLK, NT, true>), dim3(dm.n * bh), dim3(NT), 0, s, dm, a.Q, a.Qp, nullptr, nullptr,
                       dm.n, a.Kpb, dm.m, nullptr, a.Spool, a.DB, a.Mc_bits, ScoreArgs{}, 0);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gapr_keys(const Dims& dm, const GaprArgs& a, hipStream_t s) {
  if (dm.d == 128 && dm.blk == 128) return launch_gapr_keys_t<128, 128>(dm, a, s);
  if (dm.d == 128 && dm.blk == 64) return launch_gapr_keys_t<128, 64>(dm, a, s);
  if (dm.d == 64 && dm.blk == 128) return launch_gapr_keys_t<64, 128>(dm, a, s);
  return launch_gapr_keys_t<64, 64>(dm, a, s);
}

hipError_t launch_gapr_queries(const Dims& dm, const GaprArgs& a, hipStream_t s) {
  if (dm.d == 128 && dm.blk == 128) return launch_gapr_queries_t<128, 128>(dm, a, s);
  if (dm.d == 128 && dm.blk == 64) return launch_gapr_queries_t<128, 64>(dm, a, s);
  if (dm.d == 64 && dm.blk == 128) return launch_gapr_queries_t<64, 128>(dm, a, s);
  return launch_gapr_queries_t<64, 64>(dm, a, s);
}

hipError_t launch_gapr_constant(const Dims& dm, const GaprArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(fill_bits_kernel, dim3(256), dim3(256), 0, s, dm, a.Mc_bits, a.mode == 2 ? 0xffffffffu : 0u);
  return hipGetLastError();
}

}  // namespace rsa
