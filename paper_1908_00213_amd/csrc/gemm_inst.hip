// One (dtype, layout) family of GEMM kernels per object file, so the families compile in parallel.
// Built several times with -DCHN_GEMM_T=<float|bf16_raw> -DCHN_GEMM_AKC=<0|1> -DCHN_GEMM_BKC=<0|1>
// -DCHN_GEMM_NAME=<symbol>.
#include "gemm_kernel.h"
#include "gemm_split.h"
#include "gemm_split_direct.h"
#include "gemm_tiny.h"

namespace chn {
namespace gemm {

chn_status CHN_GEMM_NAME(GemmArgs &g, hipStream_t st) {
  if constexpr (sizeof(CHN_GEMM_T) == 4) {
    if (g.parts == 3) return launch_tiny<CHN_GEMM_AKC != 0, CHN_GEMM_BKC != 0>(g, st);
    if (g.parts == 2) return launch_split<2, 2, 2, CHN_GEMM_AKC != 0, CHN_GEMM_BKC != 0>(g, st);
    if constexpr (CHN_GEMM_AKC && CHN_GEMM_BKC) {
      if (g.parts == 1 && !g.direct) return launch_split<1, 1, 4, true, true>(g, st);
    }
    if (g.parts == 1) return launch_split_direct<CHN_GEMM_AKC != 0, CHN_GEMM_BKC != 0>(g, st);
  }
  return launch_layout<CHN_GEMM_T, CHN_GEMM_AKC != 0, CHN_GEMM_BKC != 0>(g, st);
}

}  // namespace gemm
}  // namespace chn
