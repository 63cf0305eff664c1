// The one-launch backward of a fully connected layer (linear_bwd.hip), as gemm.hip's entry point sees it.
#pragma once
#include "common.h"
#include "gemm_args.h"

namespace chn {
namespace gemm {

enum class LinearBwd { kApart, kTiny, kSplit, kDma };
// w: the weight gradient dv^T x, both operands along M/N, with `sums`; dx: the input gradient dv W or NULL, W along K (w_kc) or N.
// Both unsplit, on tiles of the kind's size.
chn_status launch_linear_bwd(const GemmArgs &w, const GemmArgs *dx, bool w_kc, LinearBwd kind, hipStream_t st);

// A larger product, both operands along M/N, planned as it may be, that leaves parts of the sums of A's rows or B's columns in g.sums:
// splits * tiles_n of M or splits * tiles_m of N.  Not every kernel does.
bool sums_of_large(const GemmArgs &g, int isz);
chn_status launch_with_sums(const GemmArgs &g, bool of_b, int isz, hipStream_t st);

}  // namespace gemm
}  // namespace chn
