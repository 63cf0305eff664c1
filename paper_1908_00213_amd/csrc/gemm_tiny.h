// Products with few output tiles and a short contraction: the layers of a small network at a small batch.
//
// On the tiled kernels such a product is a chain of latencies -- operands to registers, to LDS, a barrier per tile step,
// an epilogue over a tile that is mostly out of range -- on one or two workgroups.  Here a workgroup of NW waves owns 32 x 32
// of C, every wave takes every NW-th chunk of the contraction straight from memory into the registers the matrix
// instruction reads (no LDS, no barrier, all loads in flight at once), the waves' sums
// meet in LDS in wave order, and every thread finishes one or a few elements, whose epilogue inputs were fetched before the
// contraction.  Any alignment and any leading dimension: vectors are read at the address they have.
// Measured (us, tiled kernels -> here, fp32): 32x10x100 9.5 -> 4.1, 32x100x100 5.8 -> 4.4, 256x256x256 10.1 -> 6.4;
// about 3.8 of it is the launch.
#pragma once
#include "gemm_kernel.h"

namespace chn {
namespace gemm {

// Four values along k (from `k` on) of one row of an operand; what lies past K reads as zero (the last value in its place,
// dropped: no load depends on a condition, so all of a batch are in flight together).
template <bool KC>
__device__ __forceinline__ uint4 tiny_load(const float *base, int64_t ld, int row, int k, int K) {
  if constexpr (KC) {
    const float *p = base + (int64_t)row * ld;
    if (k + 4 <= K) {
      const chn_u32x4 v = *reinterpret_cast<const __attribute__((address_space(1))) chn_u32x4_any *>(reinterpret_cast<uintptr_t>(p + k));
      return make_uint4(v[0], v[1], v[2], v[3]);
    }
  }
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int at = min(k + e, K - 1);
    w[e] = global_load<uint32_t>(reinterpret_cast<uintptr_t>(KC ? base + (int64_t)row * ld + at : base + (int64_t)at * ld + row));
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = k + e < K ? w[e] : 0u;
  return make_uint4(w[0], w[1], w[2], w[3]);
}

constexpr int kTinyBatch = 8;                              // chunks of eight k per wave, all in flight at once

template <bool A_KC, bool B_KC, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_tiny_kernel(GemmArgs g) {
  constexpr int CHUNK = 8, OUT = 16 / NW;                  // k per chunk; outputs per thread
  __shared__ float part[NW][32][32];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int m0 = ((int)blockIdx.x / g.tiles_n) * 32, n0 = ((int)blockIdx.x % g.tiles_n) * 32;
  const float *A = static_cast<const float *>(g.A), *Bm = static_cast<const float *>(g.B);
  const int ra = min(m0 + r, g.M - 1), rb = min(n0 + r, g.N - 1);      // (rows past the end repeat the last one: never stored)
  const int nch = (g.K + CHUNK - 1) / CHUNK;

  // what the epilogue reads besides the product, fetched before the contraction
  float c0[OUT], bias[OUT], aux[OUT];
#pragma unroll
  for (int i = 0; i < OUT; ++i) {
    const int o = (int)threadIdx.x + i * 64 * NW, row = m0 + (o >> 5), col = n0 + (o & 31);
    c0[i] = bias[i] = aux[i] = 0.0f;
    if (row < g.M && col < g.N) {
      if (g.beta != 0.0f) c0[i] = load1(g.C, (int64_t)row * g.ldc + col, g.c_bf16);
      if (g.epi >= CHN_EPI_BIAS && g.epi <= CHN_EPI_BIAS_GELU) bias[i] = g.bias[col];
      if (g.epi == CHN_EPI_RELU_BWD || g.epi == CHN_EPI_GELU_BWD) aux[i] = load1(g.aux, (int64_t)row * g.ldaux + col, g.c_bf16);
    }
  }

  floatx16 acc[1][1];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[0][0][v] = 0.0f;
  Frags<1, 1> f[kTinyBatch];
#pragma unroll
  for (int u = 0; u < kTinyBatch; ++u)
    if (wave + u * NW < nch) {                              // (uniform over the wave)
      const int k = (wave + u * NW) * CHUNK + h * 4;
      f[u].a[0] = tiny_load<A_KC>(A, g.lda, ra, k, g.K);
      f[u].b[0] = tiny_load<B_KC>(Bm, g.ldb, rb, k, g.K);
    }
#pragma unroll
  for (int u = 0; u < kTinyBatch; ++u)
    if (wave + u * NW < nch) mma<float, 1, 1>(acc, f[u]);
#pragma unroll
  for (int v = 0; v < 16; ++v) part[wave][8 * (v >> 2) + 4 * h + (v & 3)][r] = acc[0][0][v];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < OUT; ++i) {
    const int o = (int)threadIdx.x + i * 64 * NW, row = m0 + (o >> 5), col = n0 + (o & 31);
    float s[NW];                                          // the waves' sums, added as a tree
#pragma unroll
    for (int w = 0; w < NW; ++w) s[w] = part[w][o >> 5][o & 31];
#pragma unroll
    for (int q = NW / 2; q > 0; q /= 2)
#pragma unroll
      for (int w = 0; w < q; ++w) s[w] += s[w + q];
    if (row < g.M && col < g.N) {
      float pre;
      const float x = epi_math(g, s[0], c0[i], bias[i], aux[i], &pre);
      if (g.epi == CHN_EPI_BIAS_GELU && g.pre) store1(g.pre, (int64_t)row * g.ldpre + col, g.c_bf16, pre);
      if (g.epi == CHN_EPI_BF16_COPY) store1(g.pre, (int64_t)row * g.ldpre + col, 1, x);
      store1(g.C, (int64_t)row * g.ldc + col, g.c_bf16, x);
    }
  }
}

// Four waves while one batch of loads each covers the contraction, else eight or sixteen (the planner sends K up to 1024 here).
template <bool A_KC, bool B_KC>
chn_status launch_tiny(const GemmArgs &g, hipStream_t st) {
  constexpr int kPerWave = kTinyBatch * 8;
  const dim3 grid((unsigned)(g.tiles_m * g.tiles_n));
  if (g.K <= 4 * kPerWave) hipLaunchKernelGGL((gemm_tiny_kernel<A_KC, B_KC, 4>), grid, dim3(256), 0, st, g);
  else if (g.K <= 8 * kPerWave) hipLaunchKernelGGL((gemm_tiny_kernel<A_KC, B_KC, 8>), grid, dim3(512), 0, st, g);
  else if (g.K <= 16 * kPerWave) hipLaunchKernelGGL((gemm_tiny_kernel<A_KC, B_KC, 16>), grid, dim3(1024), 0, st, g);
  else return fail(CHN_ERR_SHAPE, "gemm: K = %d is beyond the small-product kernel", g.K);
  return check_launch("gemm (tiny)");
}

}  // namespace gemm
}  // namespace chn
