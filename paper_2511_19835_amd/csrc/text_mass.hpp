// Log-masses of the text key blocks (paper Sec. 3.2, Sec. 4.1; Alg. 1 steps 5-7):
//   Lmass[n][N+i] = log sum_{t in text block i} exp(scale * q^pool_n . k_t)
// as a device function, because three launches carry it: the key side of the gate, the launch that pools V when the
// gate is off (the streaming of V is bound by HBM, this by latency and the fp32 matrix rate), and text_mass_kernel by
// itself.
#pragma once
#include "rsa_common.hpp"

namespace rsa {

constexpr int kTextQueries = 32;                                      // pooled queries per workgroup
constexpr int kTextTokens = 128;                                      // ... and text tokens: one block of 128 or two of 64
constexpr int kTextMassLdsFloats = 2 * (kTextTokens / 32) * kTextQueries;
__host__ __device__ inline int text_mass_workgroups(const Dims& dm) {  // of one (batch, head)
  return (dm.n + kTextQueries - 1) / kTextQueries * (int)((dm.tt + kTextTokens - 1) / kTextTokens);
}

// Where rsa_pool makes the text log-masses when the gate is on: with the key side of the gate, which is what lets Q and V
// be pooled in one launch, or, when there are more than two workgroups per CU of them, with the pooling of V, under whose
// streaming they cost nothing (24 heads, 512 text tokens and 512 query blocks, 1536 workgroups: the key side 218 -> 253 us
// with them, the two pooling launches 219 us against 199 as one).
inline bool text_rides_with_keys(const Dims& dm) { return (long long)text_mass_workgroups(dm) * dm.batch * dm.heads <= 512; }

// Workgroup `wg` of the text_mass_workgroups() of (batch, head) bh: 32 pooled queries against 128 text tokens, a
// wave per 32 tokens, v_mfma_f32_32x32x2_f32 (fp32 operands, products and sums; a bf16 key is exact in fp32), then
// one log-sum-exp per query and text block. A lane holds 16 scores of one query, so the block's maximum and sum go
// across the two half-waves and, through LDS, across the waves of the block. Bound by latency: one pass of loads, a
// chain of D/2 matrix instructions (2 us at d = 128) and two barriers. (A token per thread and eight queries on the
// vector ALU, the block sums then taken one query at a time by a wave, was 11 us in the smallest call, now 5; with 512
// text tokens it reached out from under the pooling of V: 165 us for the launch at 24 heads of 65 536 tokens, now 145.)
// `lds`: kTextMassLdsFloats floats.
template <int D, int BLK>
__device__ __forceinline__ void text_mass_block(const Dims& dm, const ScoreArgs& a, int wg, int bh, float* lds) {
  constexpr int TB = BLK / 32;                   // token tiles (waves) of a text block
  float (*mxs)[kTextQueries] = reinterpret_cast<float (*)[kTextQueries]>(lds);
  float (*sums)[kTextQueries] = mxs + kTextTokens / 32;
  const int b = bh / dm.heads, h = bh % dm.heads;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, l32 = lane % 32, hf = lane / 32;
  const int query_tiles = (dm.n + kTextQueries - 1) / kTextQueries;
  const int n = (wg % query_tiles) * kTextQueries + l32;
  const int t0 = (wg / query_tiles) * kTextTokens + 32 * wave;       // this wave's first text token
  const int last = (int)dm.tt - 1;
  const uint16_t* Kt = a.K + (int64_t)b * dm.sb + (int64_t)h * dm.sh + dm.tv * dm.st;
  const uint4* krow = reinterpret_cast<const uint4*>(Kt + (int64_t)(t0 + l32 < last ? t0 + l32 : last) * dm.st);
  const floatx4* qrow = reinterpret_cast<const floatx4*>(a.Qp + ((size_t)bh * dm.n + (n < dm.n ? n : dm.n - 1)) * D);
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  // A = text keys (M = token), B = pooled queries (N = query); rows past the end repeat the last one and are masked
  // (both half-waves read the whole row and take the even or the odd channels)
#pragma unroll 4
  for (int i = 0; i < D / 8; ++i) {
    const uint4 kv = krow[i];
    const floatx4 q0 = qrow[2 * i], q1 = qrow[2 * i + 1];
    const uint32_t w[4] = {kv.x, kv.y, kv.z, kv.w};
    const float q[4] = {hf ? q0[1] : q0[0], hf ? q0[3] : q0[2], hf ? q1[1] : q1[0], hf ? q1[3] : q1[2]};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bf16_bits_to_float(hf ? w[e] >> 16 : w[e] & 0xffffu), q[e], acc, 0, 0, 0);
  }
  // accumulator register r: token t0 + 8(r/4) + 4*hf + r%4, query n
  float mx = -INFINITY;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    acc[r] = t0 + 8 * (r / 4) + 4 * hf + (r % 4) <= last ? acc[r] * dm.scale : -INFINITY;
    mx = fmaxf(mx, acc[r]);
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  if (hf == 0) mxs[wave][l32] = mx;
  __syncthreads();
  const int w0 = wave / TB * TB;                 // first wave of this text block
#pragma unroll
  for (int w = 0; w < TB; ++w) mx = fmaxf(mx, mxs[w0 + w][l32]);
  float sum = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) sum += expf(acc[r] - mx);             // exp(-inf) = 0 past the end
  sum += __shfl_xor(sum, 32);
  if (hf == 0) sums[wave][l32] = sum;
  __syncthreads();
  if (wave == w0 && hf == 0 && n < dm.n && t0 <= last) {
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < TB; ++w) total += sums[w0 + w][l32];
    a.Lmass[((size_t)bh * dm.n + n) * dm.m + dm.n + t0 / BLK] = mx + logf(total);
  }
}

}  // namespace rsa
