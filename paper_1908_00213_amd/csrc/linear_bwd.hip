// chn_linear_bwd: the backward of a fully connected layer -- weight gradient, bias gradient and input gradient -- in one call and,
// where the products are small, in one launch.
//
// The two products and the column sums read the same gradient and do not depend on each other.  One after the other, each pays for its
// launch, the first trip to memory and its epilogue, and leaves most of a compute unit's waves unused meanwhile.  Here the blocks
// of both products share a grid, and the blocks of the weight gradient's first tile column add up the rows of dv^T that pass through their
// registers: the bias gradient.  Three kernels, each the body of one of chn_gemm's: the latency-bound one of gemm_tiny.h, the 64x64
// tile of gemm_split_direct.h (fp32) and of the direct-copy kernel (bfloat16).
#include "gemm_split.h"
#include "gemm_split_direct.h"
#include "gemm_tiny.h"
#include "linear_bwd.h"

namespace chn {
namespace gemm {

// The first `n_w` blocks: the weight gradient, both operands along M/N; the others: the input gradient, W along K or along N.
template <bool W_KC, int NW>
__global__ __launch_bounds__(64 * NW) void linear_bwd_tiny_kernel(GemmArgs w, GemmArgs x, int n_w) {
  __shared__ float lds[kTinyLds<16, NW>];
  if ((int)blockIdx.x < n_w) tiny_block<16, false, false, NW, true>(w, blockIdx.x, lds);
  else tiny_block<16, true, W_KC, NW, false>(x, blockIdx.x - n_w, lds);
}

template <bool W_KC>
__global__ __launch_bounds__(64 * kDirectWaves) void linear_bwd_split_kernel(GemmArgs w, GemmArgs x, int n_w) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int redo;
  if ((int)blockIdx.x < n_w) split_direct_block<false, false, Sums::kRows>(w, blockIdx.x, lds, redo);
  else split_direct_block<true, W_KC, Sums::kNone>(x, blockIdx.x - n_w, lds, redo);
}

template <bool W_KC>
__global__ __launch_bounds__(256) void linear_bwd_dma_kernel(GemmArgs w, GemmArgs x, int n_w) {
  __shared__ __align__(1024) char stage0[kSmallDmaStage<1>];
  __shared__ __align__(1024) char stage1[kSmallDmaStage<1>];
  __shared__ __align__(1024) char stage2[kSmallDmaStage<1>];
  __shared__ __align__(1024) char stage3[kSmallDmaStage<1>];
  if ((int)blockIdx.x < n_w) small_dma_block<1, false, false, Sums::kRows>(w, blockIdx.x, stage0, stage1, stage2, stage3);
  else small_dma_block<1, true, W_KC, Sums::kNone>(x, blockIdx.x - n_w, stage0, stage1, stage2, stage3);
}

namespace {

template <bool W_KC>
chn_status launch_split_pair(const GemmArgs &w, const GemmArgs &x, int n_w, int n_x, hipStream_t st) {
  auto kern = linear_bwd_split_kernel<W_KC>;
  static std::atomic<bool> configured{false};  // per instantiation
  CHN_TRY(reserve_lds(configured, reinterpret_cast<const void *>(kern), kDirectLds));
  hipLaunchKernelGGL(kern, dim3((unsigned)(n_w + n_x)), dim3(64 * kDirectWaves), kDirectLds, st, w, x, n_w);
  return check_launch("linear_bwd (split fp32)");
}

}  // namespace

chn_status launch_linear_bwd(const GemmArgs &w, const GemmArgs *dx, bool w_kc, LinearBwd kind, hipStream_t st) {
  const GemmArgs x = dx ? *dx : w;
  const int n_w = w.tiles_m * w.tiles_n, n_x = dx ? x.tiles_m * x.tiles_n : 0;
  const dim3 grid((unsigned)(n_w + n_x));
  if (kind == LinearBwd::kTiny) {
    const int nw = dx && x.K > w.K ? tiny_waves(x.K) : tiny_waves(w.K);
#define CHN_TINY(NW)                                                                                                       \
    if (w_kc) hipLaunchKernelGGL((linear_bwd_tiny_kernel<true, NW>), grid, dim3(64 * NW), 0, st, w, x, n_w);               \
    else hipLaunchKernelGGL((linear_bwd_tiny_kernel<false, NW>), grid, dim3(64 * NW), 0, st, w, x, n_w)
    if (nw == 4) { CHN_TINY(4); }
    else if (nw == 8) { CHN_TINY(8); }
    else { CHN_TINY(16); }
#undef CHN_TINY
    return check_launch("linear_bwd (tiny)");
  }
  if (kind == LinearBwd::kDma) {
    if (w_kc) hipLaunchKernelGGL((linear_bwd_dma_kernel<true>), grid, dim3(256), 0, st, w, x, n_w);
    else hipLaunchKernelGGL((linear_bwd_dma_kernel<false>), grid, dim3(256), 0, st, w, x, n_w);
    return check_launch("linear_bwd (direct copy)");
  }
  return w_kc ? launch_split_pair<true>(w, x, n_w, n_x, st) : launch_split_pair<false>(w, x, n_w, n_x, st);
}

bool sums_of_large(const GemmArgs &g, int isz) {
  if (isz == 2) return g.tile < 2 && g.dma;
  return g.parts == 1 || (g.parts == 2 && (g.piece == 16 || (g.any_a && g.any_b)));
}

template <Sums SUMS>
chn_status launch_large(const GemmArgs &g, int isz, hipStream_t st) {
  if (isz == 2) return g.tile == 1 ? launch_small_dma<2, false, false, SUMS>(g, st) : launch_small_dma<1, false, false, SUMS>(g, st);
  if (g.parts == 1) return launch_split_direct<false, false, SUMS>(g, st);
  if (g.piece == 16) return launch_split_piece<2, 2, 2, false, false, 16, 16, SUMS>(g, st);
  return launch_split_piece<2, 2, 2, false, false, kAnyPiece, kAnyPiece, SUMS>(g, st);
}
chn_status launch_with_sums(const GemmArgs &g, bool of_b, int isz, hipStream_t st) {
  return of_b ? launch_large<Sums::kColumnParts>(g, isz, st) : launch_large<Sums::kRowParts>(g, isz, st);
}

}  // namespace gemm
}  // namespace chn
