// Implicit full attention from pooled query-key interactions (paper Sec. 3.2, Sec. 4.1;
// Alg. 1 steps 5-7). Everything stays fp32: the selection that follows compares these
// values and is checked against an fp64 reference inside a 1e-4 band.
//
//   pooled_scores_kernel   Spool[n][m] = scale * q^pool_n . k^pool_m       (N x M x d, tiny)
//   text_mass_kernel       Lmass[n][N+i] = log sum_{t in text block i} exp(scale * q^pool_n . k_t)
//   ipar_softmax_rows_kernel  Lmass[n][m<N] = Spool + ln c_m ; Apool = row-softmax(Lmass)
//   ipar_fused_kernel      the first and the third in one pass (rows of at most 1024 blocks; up to 2048 where one_pass says so)
//
// softmax(Lmass) is the paper's reallocation written in log space: the mixed softmax
// over [pooled video keys ; text tokens] gives weights proportional to exp(score); a video
// block is then multiplied by its token count (exp(s + ln c)), text tokens are summed per
// block (exp(logsumexp)), and everything is divided by the row total.
#include <type_traits>

#include "lds_dma.hpp"
#include "rsa_common.hpp"
#include "text_mass.hpp"

namespace rsa {
namespace {

__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// One wave per 32 x 32 output tile, v_mfma_f32_32x32x2_f32: fp32 operands, fp32 products and
// sums, so the scores keep full single precision (the selection that follows is compared with
// fp64 inside a 1e-4 band). The contraction index may be visited in any order as long as both
// operands agree: k-step s takes channel s from the lanes of the lower half-wave and channel
// D/2 + s from the upper one, so every lane needs D/2 consecutive floats of its row.
// The 64 query rows and 64 key rows of a workgroup come in through LDS: read from global memory
// with every wave load covering two whole rows (a lane reading its own row directly touches 64
// cache lines per load and the kernel is then bound by the address unit of the CU), then read
// back per lane; a row stride of D + 4 floats keeps the 16-byte LDS reads free of bank conflicts.
template <int D>
__global__ __launch_bounds__(256) void pooled_scores_kernel(Dims dm, ScoreArgs a) {
  constexpr int KH = D / 2;                     // k-steps; channels per half-wave
  constexpr int RS = D + 4;                     // LDS row stride in floats
  constexpr int C4 = D / 4;                     // float4 per row
  __shared__ float rows[2][64 * RS];            // [0]: pooled queries n0 .. n0+63, [1]: pooled keys m0 .. m0+63
  const int bh = blockIdx.z;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int l32 = lane % 32, hf = lane / 32;
  const int nb = blockIdx.y * 64, mb = blockIdx.x * 64;
  for (int idx = threadIdx.x; idx < 64 * C4; idx += 256) {
    const int r = idx / C4, c4 = idx % C4;
    const int n = nb + r < dm.n ? nb + r : dm.n - 1;          // rows past the end repeat the last one (not stored)
    const int m = mb + r < dm.m ? mb + r : dm.m - 1;
    *reinterpret_cast<floatx4*>(&rows[0][r * RS + 4 * c4]) =
        *reinterpret_cast<const floatx4*>(a.Qp + ((size_t)bh * dm.n + n) * D + 4 * c4);
    *reinterpret_cast<floatx4*>(&rows[1][r * RS + 4 * c4]) =
        *reinterpret_cast<const floatx4*>(a.Kp + ((size_t)bh * dm.m + m) * D + 4 * c4);
  }
  __syncthreads();
  const int n0 = nb + (wave / 2) * 32, m0 = mb + (wave % 2) * 32;
  if (n0 >= dm.n || m0 >= dm.m) return;         // after the only barrier
  const floatx4* qrow = reinterpret_cast<const floatx4*>(&rows[0][((wave / 2) * 32 + l32) * RS + hf * KH]);
  const floatx4* krow = reinterpret_cast<const floatx4*>(&rows[1][((wave % 2) * 32 + l32) * RS + hf * KH]);
  floatx4 qv[KH / 4], kv[KH / 4];
#pragma unroll
  for (int i = 0; i < KH / 4; ++i) {
    qv[i] = qrow[i];
    kv[i] = krow[i];
  }
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  // A = pooled queries (M = query row), B = pooled keys (N = key column)
#pragma unroll
  for (int i = 0; i < KH / 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qv[i][e], kv[i][e], acc, 0, 0, 0);
  // accumulator register r: query row n0 + 8(r/4) + 4*hf + r%4, key column m0 + l32
  float* S = a.Spool + (size_t)bh * dm.n * dm.m;
  if (m0 + l32 < dm.m) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = n0 + 8 * (r / 4) + 4 * hf + (r % 4);
      if (row < dm.n) S[(size_t)row * dm.m + m0 + l32] = acc[r] * dm.scale;
    }
  }
}

// The text log-masses by themselves (text_mass.hpp has the work).
template <int D, int BLK>
__global__ __launch_bounds__(256) void text_mass_kernel(Dims dm, ScoreArgs a) {
  __shared__ float lds[kTextMassLdsFloats];
  text_mass_block<D, BLK>(dm, a, blockIdx.x, blockIdx.y, lds);
}

// One wave per row, the row held in registers (rows of at most 64 * NI blocks), so every value
// is read once, every exponential is taken once and no barrier is needed.
template <int NI>
__global__ __launch_bounds__(256) void ipar_softmax_rows_kernel(Dims dm, ScoreArgs a) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int n = blockIdx.x * 4 + wave, bh = blockIdx.y;
  if (n >= dm.n) return;                         // no barriers in this kernel
  const size_t row = ((size_t)bh * dm.n + n) * dm.m;
  const float* S = a.Spool + row;
  float* L = a.Lmass + row;
  float* A = a.Apool + row;
  const float ln_full = logf((float)dm.blk), ln_last = logf((float)dm.block_count(dm.n - 1));
  float l[NI];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int m = lane + 64 * i;
    l[i] = -INFINITY;
    if (m < dm.m) {
      if (m < dm.n) {
        l[i] = S[m] + (m == dm.n - 1 ? ln_last : ln_full);
        L[m] = l[i];
      } else {
        l[i] = L[m];
      }
    }
    mx = fmaxf(mx, l[i]);
  }
  mx = wave_max(mx);
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    l[i] = expf(l[i] - mx);                      // exp(-inf) = 0 for the slots past the row end
    sum += l[i];
  }
  sum = wave_sum(sum);
  const float inv = 1.0f / sum;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int m = lane + 64 * i;
    if (m < dm.m) A[m] = l[i] * inv;
  }
}

// Reduction over the 16 lanes of each row of lanes with data-parallel-primitive moves: lane 15 of every
// row ends up with the result.
template <bool MAX>
__device__ __forceinline__ float lane_row_reduce(float v) {
  constexpr int kIdentity = MAX ? (int)0xff800000u : 0;       // -inf or 0 for lanes without a source
  auto step = [&](auto ctrl) __attribute__((always_inline)) {
    const int o = __builtin_amdgcn_update_dpp(kIdentity, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, false);
    const float f = __builtin_bit_cast(float, o);
    v = MAX ? fmaxf(v, f) : v + f;
  };
  step(std::integral_constant<int, 0x111>{});   // row_shr:1
  step(std::integral_constant<int, 0x112>{});   // row_shr:2
  step(std::integral_constant<int, 0x114>{});   // row_shr:4
  step(std::integral_constant<int, 0x118>{});   // row_shr:8
  return v;
}

// Log-mass of a video block: the score as it is stored (rounded), then the logarithm of the block's token count --
// not one fused operation, so that it is the same number in every kernel that works it out.
__device__ __forceinline__ float video_log_mass(float product, float scale, float ln_count) {
#pragma clang fp contract(off)
  const float score = product * scale;
  return score + ln_count;
}

// Alg. 1 steps 5-7 in one pass over the N x M tensors (rows of at most 64 * NT blocks): a workgroup
// owns 16 pooled queries and all M key blocks, which its waves share out evenly (a band of consecutive
// columns, 16-block tiles, at most NT of them). The product is v_mfma_f32_16x16x4_f32 (fp32 operands,
// products and sums, at the rate of the 32x32x2 form), and every score of the wave's band stays in
// registers. Scores are written once (Spool), turned into log-masses (video blocks: + ln c_m; text blocks:
// what text_mass left in Lmass), and the row softmax is taken across the registers, the lanes and the four
// waves, so that Lmass and Apool are written once too and nothing is read back. The text columns of Lmass
// must be in place before this kernel runs.
//
// Sixteen rows rather than 32: four workgroups fit a CU (two for rows of 1025 to 2048 blocks), so that the
// stores of one run beside the matrix work of another and the last round of workgroups is shorter, a few
// heads fill the chip, and the scores of 2048 columns still fit the registers. Bound by the stores and the fp32
// matrix work about equally, one after the other within a round. Against 32 rows (and against a scores kernel and a
// softmax kernel for rows above 1024): 2 heads of 17 blocks 12.5 -> 5.3 us, 24 heads of 159 blocks 17 -> 12, of 516
// 72 -> 50, of 931 143 -> 111, of 1182 266 -> 222; 3 heads of 931 51 -> 36. Three or four buffers instead of two: no
// gain at any of these (latency is covered), and fewer workgroups per CU.
//
// Each wave has a piece of LDS to itself:
//  - in the product, two buffers of half a key tile: the pooled keys come in with direct-to-LDS loads,
//    the contraction index in two halves, the half after the one being multiplied always on its way. The four
//    terms of a matrix instruction, one per lane row, are channels 2s, D/2 + 2s, 2s + 1, D/2 + 2s + 1, the order in
//    which the 32x32x2 instructions of pooled_scores_kernel take them: the scores are the same bits there and
//    here. A buffer row is one key block: PPR 16-byte positions; position p of row r holds logical chunk
//    p ^ key(r), so that lanes reading one logical chunk of 16 rows hit 16 different positions;
//  - in the epilogue, a [16][16 * HT] tile of floats (rows padded by 16 bytes) through which the accumulators
//    (a lane holds one column of 4 rows) are turned into rows, so that a store instruction writes runs of
//    64 * HT bytes: a wave may have 63 stores in flight, and with narrow ones that bound, not the memory,
//    sets the pace.
typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));
template <int D, int NT>
__global__ __launch_bounds__(256, NT <= 16 ? 4 : 2) void ipar_fused_kernel(Dims dm, ScoreArgs a) {
  constexpr int KH = D / 2, KQ = D / 4;         // k-steps = channels per lane row: KQ
  constexpr int PPR = D / 8;                    // 16-byte positions per buffer row (half the channels of a key block)
  constexpr int CPH = PPR / 2;                  // ... of the channels below D/2, and of those above
  constexpr int HALF = 16 * PPR * 4;            // floats per buffer
  constexpr int RPL = 64 / PPR;                 // rows per load
  constexpr int LOADS = 16 / RPL;               // direct-to-LDS loads per half tile
  constexpr int HT = NT < 8 ? NT : 8;           // tiles per epilogue pass
  constexpr int TW = 16 * HT, TS = TW + 4;      // epilogue tile: columns, row stride in floats
  constexpr int WAVE_LDS = ((2 * HALF > 16 * TS ? 2 * HALF : 16 * TS) + 255) / 256 * 256;   // floats
  __shared__ __attribute__((aligned(1024))) float wlds[4][WAVE_LDS];
  __shared__ __attribute__((aligned(16))) float red[2][4][16];               // row maxima, then row sums, of each wave
  // Workgroups go round the 8 XCDs by their index; XCD x takes a contiguous eighth of the row tiles of all
  // (batch, head) pairs, so that the pooled keys its L2 serves at any time are those of a head or two and
  // few heads still use all XCDs.
  const int row_tiles = (dm.n + 15) / 16;
  const int total = row_tiles * dm.batch * dm.heads, q8 = total / 8, r8 = total % 8;
  const int xcd = blockIdx.x % 8;
  const int item = xcd * q8 + (xcd < r8 ? xcd : r8) + (int)blockIdx.x / 8;
  const int bh = item / row_tiles;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int l16 = lane % 16, g = lane / 16;
  const int n0 = (item % row_tiles) * 16;
  const int M = dm.m, N = dm.n;
  float* mine = wlds[wave];

  // this lane's pooled query (row n0 + l16, clamped: rows past the end are computed and not stored)
  float qv[KQ];
  {
    const int n = n0 + l16 < N ? n0 + l16 : N - 1;
    const floatx4* qrow = reinterpret_cast<const floatx4*>(a.Qp + ((size_t)bh * N + n) * D + (g % 2) * KH);
#pragma unroll
    for (int i = 0; i < KH / 4; ++i) {
      const floatx4 q = qrow[i];
      qv[2 * i] = g < 2 ? q[0] : q[1];
      qv[2 * i + 1] = g < 2 ? q[2] : q[3];
    }
  }
  // the query must be in before the first direct-to-LDS load goes out: the compiler does not see those
  // loads and would wait for them together with the query at its first use
  __builtin_amdgcn_s_waitcnt(0x0F70);           // vmcnt(0)
  floatx4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int n_tiles = (M + 15) / 16;
  const int per_wave = (n_tiles + 3) / 4;       // tiles of a band (at most NT)
  const int ct0 = wave * per_wave;
  const int my_tiles = max(0, min(per_wave, n_tiles - ct0));
  const float* Kp = a.Kp + (size_t)bh * M * D;
  const int lrow = lane / PPR, lpos = lane % PPR;
  auto swz = [](int r) __attribute__((always_inline)) { return (r / (16 / PPR)) & (PPR - 1); };
  // half u % 2 of the band's key tile u / 2 into buffer u % 2
  auto request_half = [&](int u) __attribute__((always_inline)) {
    const int m0 = (ct0 + u / 2) * 16, c = u % 2;
    const uint32_t dst = (uint32_t)(uintptr_t)(mine + (u % 2) * HALF);
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      const int r = j * RPL + lrow;
      const int m = m0 + r < M ? m0 + r : M - 1;     // rows past the end repeat the last one (not stored)
      const int q = lpos ^ swz(r);                   // logical chunk: q / CPH = channels below or above D/2, chunk q % CPH of this half
      const int ch = (q / CPH) * KH + c * (KH / 2) + 4 * (q % CPH);
      dma16_v(dst + j * 1024, Kp + (size_t)m * D + ch, &wlds[0][0]);
    }
  };
  const int halves = 2 * my_tiles;
  if (halves > 0) request_half(0);
#pragma unroll
  for (int u = 0; u < 2 * NT; ++u) {
    if (u < halves) {                            // wave-uniform
      // the buffer of the next half was last read in the step before: those reads fed MFMAs that have been issued
      if (u + 1 < halves) {
        request_half(u + 1);
        wait_loads_leaving<LOADS>();
      } else {
        wait_loads_leaving<0>();
      }
      asm volatile("" ::: "memory");             // no read of the buffer may move above the wait
      const float* kb = mine + (u % 2) * HALF + l16 * (PPR * 4) + g / 2;
#pragma unroll
      for (int i = 0; i < CPH; ++i) {
        const float* kc = kb + (((g % 2) * CPH + i) ^ swz(l16)) * 4;
        const float k0 = kc[0], k1 = kc[2];
        acc[u / 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(qv[(u % 2) * (KQ / 2) + 2 * i], k0, acc[u / 2], 0, 0, 0);
        acc[u / 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(qv[(u % 2) * (KQ / 2) + 2 * i + 1], k1, acc[u / 2], 0, 0, 0);
      }
    }
  }

  // accumulator register r of tile t: query row n0 + 4*g + r, key block 16*(ct0 + t) + l16.
  const size_t row0 = (size_t)bh * N * M;
  float* S = a.Spool + row0;
  float* L = a.Lmass + row0;
  float* A = a.Apool + row0;
  const float ln_full = logf((float)dm.blk), ln_last = logf((float)dm.block_count(N - 1));
  const int band0 = ct0 * 16, band1 = band0 + 16 * my_tiles;      // the wave's columns
  // Writes f(t, r) for every accumulator to rows n0 .. n0+15 of `out`, the band's columns below `col_end`, through
  // the wave's LDS tile: HT tiles at a time, whole rows of the tile per store.
  auto store_band = [&](float* out, int col_end, auto f) __attribute__((always_inline)) {
    const int end = col_end < band1 ? col_end : band1;
#pragma unroll
    for (int p0 = 0; p0 < NT; p0 += HT) {
      if (band0 + 16 * p0 < end) {               // wave-uniform
        asm volatile("" ::: "memory");
#pragma unroll
        for (int tt = 0; tt < HT; ++tt)
#pragma unroll
          for (int r = 0; r < 4; ++r) mine[(4 * g + r) * TS + 16 * tt + l16] = f(p0 + tt, r);
        asm volatile("" ::: "memory");
        // a tile row is TW / 4 lanes of four floats: 64 lanes take RPI rows per store instruction, U instructions
        // at a time (all 16 / RPI unrolled: their addresses would be worked out ahead and spill)
        constexpr int LPR = TW / 4, RPI = 64 / LPR < 16 ? 64 / LPR : 16, U = 16 / RPI < 4 ? 16 / RPI : 4;
        const int rsub = lane / LPR, cl = 4 * (lane % LPR);
        const int m = band0 + 16 * p0 + cl;
        const float* src = &mine[rsub * TS + cl];
        float* dst = out + (size_t)(n0 + rsub) * M + m;
#pragma clang loop unroll(disable)
        for (int i = 0; i < 16; i += U * RPI) {
          floatx4 v[U];
#pragma unroll
          for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const floatx4*>(src + u * RPI * TS);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            float* d = dst + (size_t)(u * RPI) * M;
            if (n0 + i + u * RPI + rsub < N) {
              if (m + 3 < end) {
                *reinterpret_cast<floatx4_u*>(d) = v[u];
              } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                  if (m + e < end) d[e] = v[u][e];
              }
            }
          }
          src += U * RPI * TS;
          dst += (size_t)(U * RPI) * M;
        }
      }
    }
  };
  // (the scores first, with nothing but stores in flight: a load in between would be waited for together
  // with every store before it)
  store_band(S, M, [&](int t, int r) __attribute__((always_inline)) { return acc[t][r] * dm.scale; });
  float pm[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) pm[r] = -INFINITY;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int tile_first = band0 + 16 * t, m = tile_first + l16;
    if (t < my_tiles && tile_first + 16 < N) {   // wave-uniform: video blocks only, none of them the last
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc[t][r] = video_log_mass(acc[t][r], dm.scale, ln_full);
        pm[r] = fmaxf(pm[r], acc[t][r]);
      }
    } else if (t < my_tiles) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int n = n0 + 4 * g + r;
        float l = -INFINITY;
        if (m < N) l = video_log_mass(acc[t][r], dm.scale, m == N - 1 ? ln_last : ln_full);
        else if (m < M) l = L[(size_t)(n < N ? n : N - 1) * M + m];
        acc[t][r] = l;
        pm[r] = fmaxf(pm[r], l);
      }
    }
  }
  // the log-masses of the video blocks (the text columns already hold theirs)
  store_band(L, N, [&](int t, int r) __attribute__((always_inline)) { return acc[t][r]; });
  // row maxima: over the lanes of the lane row, then over the waves through LDS
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float v = lane_row_reduce<true>(pm[r]);
    if (l16 == 15) red[0][wave][4 * g + r] = v;
  }
  __syncthreads();
  floatx4 mx = *reinterpret_cast<const floatx4*>(&red[0][0][4 * g]);
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    const floatx4 u = *reinterpret_cast<const floatx4*>(&red[0][w][4 * g]);
#pragma unroll
    for (int e = 0; e < 4; ++e) mx[e] = fmaxf(mx[e], u[e]);
  }
  float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (t < my_tiles) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float e = expf(acc[t][r] - mx[r]);    // exp(-inf) = 0 for the columns past the row end
        acc[t][r] = e;
        ps[r] += e;
      }
    }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float v = lane_row_reduce<false>(ps[r]);
    if (l16 == 15) red[1][wave][4 * g + r] = v;
  }
  __syncthreads();
  floatx4 inv = *reinterpret_cast<const floatx4*>(&red[1][0][4 * g]);
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    const floatx4 u = *reinterpret_cast<const floatx4*>(&red[1][w][4 * g]);
#pragma unroll
    for (int e = 0; e < 4; ++e) inv[e] += u[e];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) inv[e] = 1.0f / inv[e];
  store_band(A, M, [&](int t, int r) __attribute__((always_inline)) { return acc[t][r] * inv[r]; });
}

// Rows of 1025 to 2048 blocks keep 32 tiles in registers, two workgroups to a CU: a round of 512, and with few heads a
// last round that is mostly empty costs more than the pass over the scores that is saved. In one pass at d = 128 where
// the rounds are at least 17/20 full; at d = 64, where the product is half as long, not at all. rsa_pool without the
// gate, us, two kernels and one pass, d = 128: 1 head of 1030 blocks of 64 37 and 58, 8 heads of 1182 227 and 259, 6 of 1182
// (444 workgroups) 171 and 168, 24 of 1182 (1776) 654 and 611, 8 of 2040 (1024) 518 and 442, 6 of 1400 (528) 211 and 250;
// d = 64: 24 of 1030 317 and 329, 6 of 1500 136 and 165, 24 of 1182 384 and 380.
template <int D>
bool one_pass(const Dims& dm) {
  if (dm.m <= 1024) return true;
  const long long round = 512, wgs = (long long)((dm.n + 15) / 16) * dm.batch * dm.heads, rounds = (wgs + round - 1) / round;
  return D == 128 && dm.m <= 2048 && 20 * wgs >= 17 * rounds * round;
}

template <int D, int BLK>
hipError_t launch_scores_t(const Dims& dm, const ScoreArgs& a, hipStream_t s) {
  const int bh = dm.batch * dm.heads;
  if (one_pass<D>(dm)) {
    // the text log-masses first, then one pass
    if (dm.tt > 0 && !a.text_done)
      hipLaunchKernelGGL((text_mass_kernel<D, BLK>), dim3(text_mass_workgroups(dm), bh), dim3(256), 0, s, dm, a);
    const dim3 fgrid(bh * ((dm.n + 15) / 16));
    if (dm.m <= 128)
      hipLaunchKernelGGL((ipar_fused_kernel<D, 2>), fgrid, dim3(256), 0, s, dm, a);
    else if (dm.m <= 256)
      hipLaunchKernelGGL((ipar_fused_kernel<D, 4>), fgrid, dim3(256), 0, s, dm, a);
    else if (dm.m <= 512)
      hipLaunchKernelGGL((ipar_fused_kernel<D, 8>), fgrid, dim3(256), 0, s, dm, a);
    else if (dm.m <= 1024)
      hipLaunchKernelGGL((ipar_fused_kernel<D, 16>), fgrid, dim3(256), 0, s, dm, a);
    else if constexpr (D == 128)
      hipLaunchKernelGGL((ipar_fused_kernel<D, 32>), fgrid, dim3(256), 0, s, dm, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((pooled_scores_kernel<D>), dim3((dm.m + 63) / 64, (dm.n + 63) / 64, bh), dim3(256), 0, s, dm, a);
  if (dm.tt > 0 && !a.text_done)
    hipLaunchKernelGGL((text_mass_kernel<D, BLK>), dim3(text_mass_workgroups(dm), bh), dim3(256), 0, s, dm, a);
  const dim3 rgrid((dm.n + 3) / 4, bh);
  if (dm.m <= 2048)
    hipLaunchKernelGGL(ipar_softmax_rows_kernel<32>, rgrid, dim3(256), 0, s, dm, a);
  else
    hipLaunchKernelGGL(ipar_softmax_rows_kernel<RSA_MAX_BLOCKS / 64>, rgrid, dim3(256), 0, s, dm, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_scores(const Dims& dm, const ScoreArgs& a, hipStream_t s) {
  if (dm.d == 128 && dm.blk == 128) return launch_scores_t<128, 128>(dm, a, s);
  if (dm.d == 128 && dm.blk == 64) return launch_scores_t<128, 64>(dm, a, s);
  if (dm.d == 64 && dm.blk == 128) return launch_scores_t<64, 128>(dm, a, s);
  return launch_scores_t<64, 64>(dm, a, s);
}

}  // namespace rsa
