// fp32 products on the bfloat16 matrix cores, 64x64 tile: operands straight from memory to the registers that are multiplied.
//
// The scheme is gemm_split.h's (three bfloat16 parts a value, six products, scaled, odd waves with the other sign, sums that are not
// finite taken again on the fp32 instruction).  What differs is who multiplies what.  Eight waves share the contraction, a wave owns
// the whole 64x64 tile for every eighth 16 k: it loads the 128 rows' k itself, splits them in its registers and multiplies; no
// LDS and no barrier before the waves' sums meet at the end.  Through LDS a wave of the same tile owns 32x32 and reads 1 KB for every
// matrix instruction, all that LDS delivers, between barriers.  What bounds it now is the stream of operand tiles out of the L2s
// (32 KB for 64 k, 0.9 us) and, where an operand lies along K, that a load instruction touches 32 lines for 1 KB: with both along K and
// a long K the tile through LDS stays (1024x1000x1000 22 and 24-26).  Operands at any address and of any extent.  us, through LDS -> here:
// 1024x1000x784 along M/N 20.1 -> 16.9, mixed 22.6 and 21.4 -> 18.9 and 18.5, along K 18.7 -> 18.9; 1024x1024x4096 76 -> 65, mixed
// 89 and 83 -> 75 and 73; 300x200x100 7.2 -> 5.9.  Built beside it without effect: a wave's priority raised while it splits or
// multiplies, half of the waves started later, the split in stages of independent instructions.
#pragma once
#include "gemm_kernel.h"
#include "split.h"

namespace chn {
namespace gemm {

constexpr int kDirectWaves = 8, kDirectLds = 4 * kDirectWaves * 4096;      // the waves' sums: 32x32 blocks

// What a lane holds of 32 rows (columns) of an operand for 16 k: row `lane % 32`, k 4 h .. 4 h + 3 and 8 + 4 h .. of the slice.
template <bool KC> struct DirectRows {
  const float *p;                                         // the row's first element (KC), or the first row's at the lane's column
  int64_t ld;
  __device__ __forceinline__ void init(const float *base, int64_t ld_, int row, int rows_total, int h) {
    const int at = min(row, rows_total - 1);              // (rows past the end repeat the last one: they feed what is not stored)
    ld = ld_;
    p = KC ? base + at * ld + 4 * h : base + at + 4 * h * ld;
  }
  __device__ __forceinline__ void load(f32x4 (&v)[2], int k) const {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if constexpr (KC) {
        v[e] = load4f(p + k + 8 * e);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[e][i] = global_load<float>(reinterpret_cast<uintptr_t>(p + (k + 8 * e + i) * ld));
      }
    }
  }
  // the slice that the end of the contraction cuts: what lies past K reads as zero
  __device__ __forceinline__ void load_last(f32x4 (&v)[2], int k, int K, int h) const {
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int at = k + 8 * e + i, back = max(at + 4 * h - (K - 1), 0);
        const float x = global_load<float>(reinterpret_cast<uintptr_t>(KC ? p + (at - back) : p + (at - back) * ld));
        v[e][i] = back == 0 ? x : 0.0f;
      }
  }
};

// The three parts of eight values, as the matrix instruction reads them.
struct DirectParts {
  uint4 p[3];
  __device__ __forceinline__ void set(const f32x4 (&v)[2], float scale) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = v[e >> 1][2 * (e & 1)] * scale, y = v[e >> 1][2 * (e & 1) + 1] * scale;
      split2(x, y, (&p[0].x)[e], (&p[1].x)[e], (&p[2].x)[e]);
    }
  }
};

// Block `block` of the product, and its share of the sums.
template <bool A_KC, bool B_KC, Sums SUMS>
__device__ __forceinline__ void split_direct_block(const GemmArgs &g, unsigned block, char *lds, int &redo) {
  const TilePos tp = tile_pos(g, block);
  const int split = tp.split, m0 = tp.tm * 64, n0 = tp.tn * 64;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int nk_all = (g.K + 63) / 64, per_split = split_steps(g, nk_all);    // (cuts at whole steps of 64 k, as planned)
  const int end = min(g.K, (split + 1) * per_split * 64), full = end / 16;               // slices that are whole
  if (threadIdx.x == 0) redo = 0;

  DirectRows<A_KC> ra[2];
  DirectRows<B_KC> rb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    ra[i].init(static_cast<const float *>(g.A), g.lda, m0 + 32 * i + r, g.M, h);
    rb[i].init(static_cast<const float *>(g.B), g.ldb, n0 + 32 * i + r, g.N, h);
  }
  floatx16 acc[2][2], low[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.0f;
  constexpr bool kSums = SUMS != Sums::kNone, kSumB = SUMS == Sums::kColumnParts;
  const bool sums = kSums && g.sums && (SUMS != Sums::kRows || tp.tn == 0);
  const int sharing = SUMS == Sums::kRowParts ? g.tiles_n : kSumB ? g.tiles_m : 1, share = SUMS == Sums::kRowParts ? tp.tn : kSumB ? tp.tm : 0;
  float sum[2] = {0.0f, 0.0f};

  const float scale = wave & 1 ? -kSplitScale : kSplitScale;
  f32x4 va[2][2], vb[2][2];
  auto load = [&](int s) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) { ra[i].load(va[i], s * 16); rb[i].load(vb[i], s * 16); }
  };
  auto multiply = [&](int s, int next) __attribute__((always_inline)) {
    DirectParts a[2], b[2];
    if constexpr (kSums) {
      if (sums && s % sharing == share) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const f32x4 t = kSumB ? vb[i][0] + vb[i][1] : va[i][0] + va[i][1];
          sum[i] += (t[0] + t[1]) + (t[2] + t[3]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) { a[i].set(va[i], scale); b[i].set(vb[i], kSplitScale); }
    __builtin_amdgcn_sched_barrier(0);
    if (next >= 0) load(next);
    __builtin_amdgcn_sched_barrier(0);
    auto product = [&](floatx16 (&d)[2][2], int pa, int pb) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          d[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i].p[pa]), __builtin_bit_cast(bf16x8, b[j].p[pb]), d[i][j], 0, 0, 0);
    };
    product(low, 1, 1);
    product(low, 1, 0);
    product(low, 0, 1);
    product(acc, 0, 0);
    product(low, 2, 0);
    product(low, 0, 2);
  };
  const int s0 = split * per_split * 4 + wave;
  if (s0 < full) load(s0);
#pragma unroll 1
  for (int s = s0; s < full; s += kDirectWaves) multiply(s, s + kDirectWaves < full ? s + kDirectWaves : -1);
  if (split * per_split * 64 < end && full * 16 < end && (full - split * per_split * 4) % kDirectWaves == wave) {
#pragma unroll
    for (int i = 0; i < 2; ++i) { ra[i].load_last(va[i], full * 16, g.K, h); rb[i].load_last(vb[i], full * 16, g.K, h); }
    multiply(full, -1);
  }

  // The waves' sums meet in LDS: [32x32 block][wave][four values of a lane]; wave w < 4 adds up block w.
  const float unscale = (wave & 1 ? -1.0f : 1.0f) / (kSplitScale * kSplitScale);
  f32x4 *const meet = reinterpret_cast<f32x4 *>(lds);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = (acc[i][j][4 * v + e] + low[i][j][4 * v + e]) * unscale;
        meet[(((2 * i + j) * kDirectWaves + wave) * 4 + v) * 64 + lane] = x;
      }
  __syncthreads();
  const int wm = (wave >> 1) & 1, wn = wave & 1;
  floatx16 out[1][1];
  if (wave < 4) {
    float bad = 0.0f;                                     // 0, or NaN: of rows and columns that are C's
    const int rows = n0 + wn * 32 + r < g.N ? g.M - m0 - wm * 32 - 4 * h : 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      f32x4 x = meet[(wave * kDirectWaves * 4 + v) * 64 + lane];
#pragma unroll
      for (int w = 1; w < kDirectWaves; ++w) x += meet[((wave * kDirectWaves + w) * 4 + v) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        out[0][0][4 * v + e] = x[e];
        bad = 8 * v + e < rows ? __builtin_fmaf(x[e], 0.0f, bad) : bad;
      }
    }
    if (bad != 0.0f) redo = 1;
  }
  __syncthreads();
  if constexpr (kSums) {
    if (sums) {                                           // (uniform over the workgroup)
      float *part = reinterpret_cast<float *>(lds);       // [wave][half][64 rows]
#pragma unroll
      for (int i = 0; i < 2; ++i) part[(wave * 2 + h) * 64 + 32 * i + r] = sum[i];
      __syncthreads();
      const int first = kSumB ? n0 : m0, extent = kSumB ? g.N : g.M;
      if (wave == 0 && first + lane < extent) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < 2 * kDirectWaves; ++w) t += part[w * 64 + lane];
        g.sums[(int64_t)(split * sharing + share) * extent + first + lane] = t;
      }
      __syncthreads();
    }
  }
  if (redo) {
    // Some sum of this tile is not finite, with the scaled operands or at all: four waves multiply the tile again on the fp32 matrix
    // instruction, without ceremony (128 rows of 128 bytes, loaded element by element, stored, multiplied).
    TileLoader<float, 64, A_KC, 4> la;
    TileLoader<float, 64, B_KC, 4> lb;
    la.init(static_cast<const float *>(g.A), g.lda, g.M, m0, g.K);
    lb.init(static_cast<const float *>(g.B), g.ldb, g.N, n0, g.K);
    const int rp = lds_row<float>(r), sw = (r >> 1) & 7;
#pragma unroll
    for (int v = 0; v < 16; ++v) out[0][0][v] = 0.0f;
#pragma unroll 1
    for (int k0 = split * per_split * 64; k0 < end; k0 += 32) {
      if (wave < 4) { la.issue(k0); lb.issue(k0); }
      __syncthreads();
      if (wave < 4) { la.store(lds, k0); lb.store(lds + 64 * 128, k0); }
      __syncthreads();
      if (wave < 4) {
        Frags<1, 1> f;
#pragma unroll 1
        for (int ks = 0; ks < 4; ++ks) {
          f.read(lds + (wm * 32 + rp) * 128, lds + 64 * 128 + (wn * 32 + rp) * 128, ((ks * 2 + h) ^ sw) << 4);
          mma<float, 1, 1>(out, f);
        }
      }
    }
    __syncthreads();
  }
  if (wave >= 4) return;
  write_out<1, 1>(g, out, lds + wave * kEpiStageBytes<1, 1>, m0, n0, split);
}

template <bool A_KC, bool B_KC, Sums SUMS>
__global__ __launch_bounds__(64 * kDirectWaves) void gemm_split_direct_kernel(GemmArgs g) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int redo;
  split_direct_block<A_KC, B_KC, SUMS>(g, blockIdx.x, lds, redo);
}

template <bool A_KC, bool B_KC, Sums SUMS = Sums::kNone>
chn_status launch_split_direct(const GemmArgs &g, hipStream_t st) {
  auto kern = gemm_split_direct_kernel<A_KC, B_KC, SUMS>;
  static std::atomic<bool> configured{false};  // per instantiation
  CHN_TRY(reserve_lds(configured, reinterpret_cast<const void *>(kern), kDirectLds));
  hipLaunchKernelGGL(kern, dim3((unsigned)(g.tiles_m * g.tiles_n * g.splits)), dim3(64 * kDirectWaves), kDirectLds, st, g);
  CHN_TRY(check_launch("gemm (split fp32, 64x64)"));
  if (g.splits > 1) {
    const int64_t n = (int64_t)g.M * (g.ldp / 4);
    hipLaunchKernelGGL(gemm_splitk_finish_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g);
    return check_launch("gemm split-K finish");
  }
  return CHN_OK;
}

}  // namespace gemm
}  // namespace chn
