// Products with few output tiles and a short contraction: the layers of a small network at a small batch.
//
// On the tiled kernels such a product is a chain of latencies -- operands to registers, to LDS, a barrier per tile step,
// an epilogue over a tile that is mostly out of range -- on one or two workgroups.  Here a workgroup of NW waves owns TS x TS
// of C, every wave takes every NW-th chunk of the contraction straight from memory into the registers the matrix
// instruction reads (no LDS, no barrier, all loads in flight at once), the waves' sums
// meet in LDS in wave order, and every thread finishes one or a few elements, whose epilogue inputs were fetched before the
// contraction.  Any alignment and any leading dimension: vectors are read at the address they have.
// What bounds it is one trip to memory, the code's own way into the instruction cache and a dozen matrix instructions.  So
// the blocks are 16x16 where few of them are needed (a quarter of the serial matrix work of 32x32, four times as many compute units
// that pull operands), only the chunk that the end of K cuts is loaded with conditions, and the kernel is 2.5 to 4.5 KB of code, 10 KB as it was
// with conditions on every chunk and both storage types in the epilogue.  us, before -> now: 32x100x784 8.0 -> 3.9, 32x100x100
// 4.0 -> 2.5, 100x784x32 both along M/N 3.6 -> 2.5, 256x256x256 5.6 -> 3.2; an empty kernel in the same place takes 1.5.
#pragma once
#include "gemm_kernel.h"

namespace chn {
namespace gemm {

// The matrix instruction of a TS x TS block: what a lane holds of the operands (row `r`, four consecutive k from 4 q on of every
// chunk of 4 Q) and of the result (value v is row 4 q + v, by blocks of 4 Q rows, column r).
template <int TS> struct TinyTile;
template <> struct TinyTile<32> {
  static constexpr int Q = 2, V = 16;
  typedef floatx16 Acc;
  static __device__ __forceinline__ void mma(Acc &c, float a, float b) { c = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
};
template <> struct TinyTile<16> {
  static constexpr int Q = 4, V = 4;
  typedef f32x4 Acc;
  static __device__ __forceinline__ void mma(Acc &c, float a, float b) { c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

// Four values along k (from `k` on) of one row of an operand, all of which exist.
template <bool KC>
__device__ __forceinline__ f32x4 tiny_load(const float *base, int64_t ld, int row, int k) {
  if constexpr (KC) return load4f(base + (int64_t)row * ld + k);
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = global_load<float>(reinterpret_cast<uintptr_t>(base + (int64_t)(k + e) * ld + row));
  return v;
}
// The same of the chunk that the end of the contraction cuts; what lies past K reads as zero.
template <bool KC>
__device__ __forceinline__ f32x4 tiny_load_last(const float *base, int64_t ld, int row, int k, int K) {
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int at = min(k + e, K - 1);
    v[e] = global_load<float>(reinterpret_cast<uintptr_t>(KC ? base + (int64_t)row * ld + at : base + (int64_t)at * ld + row));
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = k + e < K ? v[e] : 0.0f;
  return v;
}

constexpr int kTinyPerWave = 64;                           // k per wave, all in flight at once
template <int TS> constexpr int kTinyPart = TS * TS + 16 * (TS / 4 - 1);                 // floats of a wave's sums
template <int TS, int NW> constexpr int kTinyLds = NW * (kTinyPart<TS> + 64);            // ... of all of them, and of row sums

// Block `block` of the product (SUMS: and the row sums of A, by the blocks of the first tile column).  lds: kTinyLds<TS, NW> floats.
template <int TS, bool A_KC, bool B_KC, int NW, bool SUMS>
__device__ __forceinline__ void tiny_block(const GemmArgs &g, int block, float *lds) {
  using Tile = TinyTile<TS>;
  constexpr int Q = Tile::Q, CHUNK = 4 * Q, BATCH = kTinyPerWave / CHUNK;
  constexpr int NT = 64 * NW, OUT = TS * TS > NT ? TS * TS / NT : 1, PART = kTinyPart<TS>;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & (TS - 1), q = lane / TS;
  const int tm = divide(block, g.tiles_n, g.per_column), tn = block - tm * g.tiles_n, m0 = tm * TS, n0 = tn * TS;
  const float *A = static_cast<const float *>(g.A), *Bm = static_cast<const float *>(g.B);
  const int ra = min(m0 + r, g.M - 1), rb = min(n0 + r, g.N - 1);      // (rows past the end repeat the last one: never stored)
  const int full = g.K / CHUNK;

  f32x4 a[BATCH], b[BATCH], a_last, b_last;
#pragma unroll
  for (int u = 0; u < BATCH; ++u)
    if (wave + u * NW < full) {                             // (uniform over the wave)
      const int k = (wave + u * NW) * CHUNK + q * 4;
      a[u] = tiny_load<A_KC>(A, g.lda, ra, k);
      b[u] = tiny_load<B_KC>(Bm, g.ldb, rb, k);
    }
  const bool last = full * CHUNK < g.K && full % NW == wave;
  if (last) {
    a_last = tiny_load_last<A_KC>(A, g.lda, ra, full * CHUNK + q * 4, g.K);
    b_last = tiny_load_last<B_KC>(Bm, g.ldb, rb, full * CHUNK + q * 4, g.K);
  }
  // what the epilogue reads besides the product
  float c0[OUT], bias[OUT], aux[OUT];
#pragma unroll
  for (int i = 0; i < OUT; ++i) {
    const int o = (int)threadIdx.x + i * NT, row = m0 + o / TS, col = n0 + (o & (TS - 1));
    c0[i] = bias[i] = aux[i] = 0.0f;
    if ((TS * TS >= NT || wave < TS * TS / 64) && row < g.M && col < g.N) {
      if (g.beta != 0.0f) c0[i] = static_cast<const float *>(g.C)[(int64_t)row * g.ldc + col];
      if (g.epi >= CHN_EPI_BIAS && g.epi <= CHN_EPI_BIAS_GELU) bias[i] = g.bias[col];
      if (g.epi == CHN_EPI_RELU_BWD || g.epi == CHN_EPI_GELU_BWD) aux[i] = static_cast<const float *>(g.aux)[(int64_t)row * g.ldaux + col];
    }
  }

  constexpr int CHAINS = TS == 16 ? 2 : 1;                  // (two where the registers are there: shorter ones, rounded half as often)
  typename Tile::Acc acc[CHAINS];
#pragma unroll
  for (int i = 0; i < CHAINS; ++i)
#pragma unroll
    for (int v = 0; v < Tile::V; ++v) acc[i][v] = 0.0f;
  float sum = 0.0f;
  const bool summing = SUMS && g.sums && tn == 0;
  auto multiply = [&](const f32x4 &x, const f32x4 &y) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) Tile::mma(acc[e % CHAINS], x[e], y[e]);
    if (SUMS && summing) sum += (x[0] + x[1]) + (x[2] + x[3]);
  };
#pragma unroll
  for (int u = 0; u < BATCH; ++u)
    if (wave + u * NW < full) multiply(a[u], b[u]);
  if (last) multiply(a_last, b_last);
  // (sixteen floats between groups of four rows: the lanes of a result's Q row groups write to different banks)
  auto at = [](int row, int col) { return row * TS + col + (row >> 2) * 16; };
#pragma unroll
  for (int v = 0; v < Tile::V; ++v) lds[wave * PART + at(4 * Q * (v >> 2) + 4 * q + (v & 3), r)] = CHAINS == 2 ? acc[0][v] + acc[CHAINS - 1][v] : acc[0][v];
  float *const sums = lds + NW * PART;
  if (SUMS && summing) sums[wave * 64 + lane] = sum;
  __syncthreads();
  if (TS * TS < NT && wave >= TS * TS / 64) return;
#pragma unroll
  for (int i = 0; i < OUT; ++i) {
    const int o = (int)threadIdx.x + i * NT, row = o / TS, col = o & (TS - 1);
    float s[NW];                                          // the waves' sums, added as a tree
#pragma unroll
    for (int w = 0; w < NW; ++w) s[w] = lds[w * PART + at(row, col)];
#pragma unroll
    for (int h = NW / 2; h > 0; h /= 2)
#pragma unroll
      for (int w = 0; w < h; ++w) s[w] += s[w + h];
    if (m0 + row < g.M && n0 + col < g.N) {
      const int64_t ci = (int64_t)(m0 + row) * g.ldc + n0 + col;
      float x = g.alpha * s[0];
      if (g.beta != 0.0f) x += g.beta * c0[i];
      x += bias[i];
      if (g.epi == CHN_EPI_BIAS_RELU) {
        x = fmaxf(x, 0.0f);
      } else if (g.epi == CHN_EPI_BIAS_GELU) {
        if (g.pre) static_cast<float *>(g.pre)[(int64_t)(m0 + row) * g.ldpre + n0 + col] = x;
        x = gelu_epi_f(x);
      } else if (g.epi == CHN_EPI_RELU_BWD) {
        x = aux[i] > 0.0f ? x : 0.0f;
      } else if (g.epi == CHN_EPI_GELU_BWD) {
        x *= gelu_grad_epi_f(aux[i]);
      } else if (g.epi == CHN_EPI_BF16_COPY) {
        static_cast<bf16_raw *>(g.pre)[(int64_t)(m0 + row) * g.ldpre + n0 + col] = f32_to_bf16(x);
      }
      static_cast<float *>(g.C)[ci] = x;
    }
  }
  if (SUMS && summing && wave == 0) {
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += sums[w * 64 + lane];
#pragma unroll
    for (int o = TS; o < 64; o *= 2) t += __shfl_xor(t, o, 64);
    if (lane < TS && m0 + lane < g.M) g.sums[m0 + lane] = t;
  }
}

template <int TS, bool A_KC, bool B_KC, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_tiny_kernel(GemmArgs g) {
  __shared__ float lds[kTinyLds<TS, NW>];
  tiny_block<TS, A_KC, B_KC, NW, false>(g, blockIdx.x, lds);
}

// Waves of a workgroup: four while one batch of loads each covers the contraction, else eight or sixteen.
inline int tiny_waves(int K) { return K <= 4 * kTinyPerWave ? 4 : K <= 8 * kTinyPerWave ? 8 : 16; }

template <int TS, bool A_KC, bool B_KC>
chn_status launch_tiny_tile(const GemmArgs &g, hipStream_t st) {
  const dim3 grid((unsigned)(g.tiles_m * g.tiles_n));
  const int nw = tiny_waves(g.K);
  if (nw == 4) hipLaunchKernelGGL((gemm_tiny_kernel<TS, A_KC, B_KC, 4>), grid, dim3(256), 0, st, g);
  else if (nw == 8) hipLaunchKernelGGL((gemm_tiny_kernel<TS, A_KC, B_KC, 8>), grid, dim3(512), 0, st, g);
  else hipLaunchKernelGGL((gemm_tiny_kernel<TS, A_KC, B_KC, 16>), grid, dim3(1024), 0, st, g);
  return check_launch("gemm (tiny)");
}
template <bool A_KC, bool B_KC>
chn_status launch_tiny(const GemmArgs &g, hipStream_t st) {
  return g.small == 16 ? launch_tiny_tile<16, A_KC, B_KC>(g, st) : launch_tiny_tile<32, A_KC, B_KC>(g, st);
}

}  // namespace gemm
}  // namespace chn
