// chn_gemm: host side of the dense product -- validation, layout classification and dispatch to the
// kernel families in gemm_kernel.h (one object file per dtype and operand layout).
#include <algorithm>
#include <atomic>
#include <utility>

#include "common.h"
#include "gemm_args.h"
#include "linear_bwd.h"

namespace chn {
namespace gemm {

#define CHN_DECL(name) chn_status name(GemmArgs &g, hipStream_t st);
CHN_DECL(launch_f32_kk) CHN_DECL(launch_f32_km) CHN_DECL(launch_f32_mk) CHN_DECL(launch_f32_mm)
CHN_DECL(launch_bf16_kk) CHN_DECL(launch_bf16_km) CHN_DECL(launch_bf16_mk) CHN_DECL(launch_bf16_mm)
#undef CHN_DECL

}  // namespace gemm
}  // namespace chn

namespace chn {
namespace {

using gemm::GemmArgs;

// chn_gemm_plan_override: what tests force instead of the planner's choice (-1: not forced)
std::atomic<int> g_force_tile{-1}, g_force_splits{-1}, g_force_direct{-1};
constexpr double kNarrowStep = 0.92, kNarrowFixed = 12.0;   // microseconds per tile step / per block of the 256 x 128 tile
constexpr int64_t kMaxLd = 1 << 22;    // fp32 products off the fp32 tiles: 32-bit byte offsets inside a tile
std::atomic<int> g_force_w8{-1};
std::atomic<int> g_force_parts{-1};   // 1: fp32 products on the three-part kernel, on the forced tile

// Largest load piece (bytes) that is aligned for every row start of the operand and divides its
// extent along the unit-stride dimension, so that a piece is never partly out of range.
// overhang: the extent need not be a multiple of the piece.  The last piece of a row then also brings
// what follows the row in memory (the padding of a pitched row, or the next row's first elements;
// never another page: the piece is aligned to its own size).  That is harmless exactly where the
// unit stride runs along M or N: those values become rows of A (columns of B) beyond M (N), and
// the rows (columns) of C they feed are never stored.
int piece_bytes(const void *p, int64_t ld_elems, int64_t extent_elems, int isz, bool overhang) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(p);
  const int64_t ldb = ld_elems * isz, ext = extent_elems * isz;
  if (a % 16 == 0 && ldb % 16 == 0 && (overhang || ext % 16 == 0)) return 16;
  if (a % 8 == 0 && ldb % 8 == 0 && (overhang || ext % 8 == 0)) return 8;
  return isz;
}

// Operand layouts (which dimension has unit stride), leading dimensions and load piece size.
chn_status classify(const chn_array *A, const chn_array *B, GemmArgs *g, bool *a_kc, bool *b_kc) {
  const int isz = dtype_size(A->dtype);
  const int64_t M = A->shape[0], K = A->shape[1], N = B->shape[1];
  auto unit = [&](const chn_array *X, int d) { return X->shape[d] <= 1 || X->strides[d] == isz; };
  if (unit(A, 1)) { *a_kc = true; g->lda = M > 1 ? A->strides[0] / isz : K; }
  else if (unit(A, 0)) { *a_kc = false; g->lda = K > 1 ? A->strides[1] / isz : M; }
  else return fail(CHN_ERR_STRIDE, "gemm: A needs a unit-stride dimension");
  if (unit(B, 0)) { *b_kc = true; g->ldb = N > 1 ? B->strides[1] / isz : K; }
  else if (unit(B, 1)) { *b_kc = false; g->ldb = K > 1 ? B->strides[0] / isz : N; }
  else return fail(CHN_ERR_STRIDE, "gemm: B needs a unit-stride dimension");
  if ((*a_kc && M > 1 && g->lda < K) || (!*a_kc && K > 1 && g->lda < M) || (*b_kc && N > 1 && g->ldb < K) || (!*b_kc && K > 1 && g->ldb < N))
    return fail(CHN_ERR_STRIDE, "gemm: overlapping (broadcast) operand rows are not supported");
  const int pa = piece_bytes(A->data, g->lda, *a_kc ? K : M, isz, false);
  const int pb = piece_bytes(B->data, g->ldb, *b_kc ? K : N, isz, false);
  g->piece_exact = pa < pb ? pa : pb;
  // the kernels that stage operands in registers take pieces that hang over the end of a row of an
  // operand whose unit stride runs along M or N
  const int qa = piece_bytes(A->data, g->lda, *a_kc ? K : M, isz, !*a_kc);
  const int qb = piece_bytes(B->data, g->ldb, *b_kc ? K : N, isz, !*b_kc);
  g->piece = qa < qb ? qa : qb;
  g->piece_a = qa; g->piece_b = qb;
  g->any_a = (*a_kc ? K : M) * isz >= 16;
  g->any_b = (*b_kc ? K : N) * isz >= 16;
  if (K == 0) { *a_kc = *b_kc = true; g->piece = g->piece_exact = g->piece_a = g->piece_b = isz; g->any_a = g->any_b = 0; }  // nothing to multiply: every load is redirected to zeros
  g->M = (int)M; g->N = (int)N; g->K = (int)K;
  return CHN_OK;
}

// Whether the direct-copy 256x256 kernel can take the product: it needs 16-byte pieces (so K is a
// multiple of the chunk length for K-contiguous operands) and 32-bit offsets inside a tile; fp32 needs
// at least one K-contiguous operand for it.
bool direct_copy_fits(const GemmArgs &g, int isz, bool a_kc, bool b_kc) {
  const bool dma_on = g_force_direct.load(std::memory_order_relaxed) != 0;
  const int64_t max_ld = (int64_t)0xffffffffu / (256 * isz);
  return dma_on && g.piece_exact == 16 && g.K > 0 && g.lda < max_ld && g.ldb < max_ld && (isz == 2 || a_kc || b_kc);
}

// Macro tile (3: 256x128, 2: 256x256, 1: 128x128, 0: 64x64) and number of K splits, chosen by a small cost model
// from measured figures: every compute unit works through its share of the blocks one after another,
// a block costing a fixed part (launch, prologue, epilogue) plus its tile steps times the time one
// compute unit needs per tile step of that tile and kernel (for the smaller tiles, of which several
// run on a compute unit at once, the amortised figure).  A problem with too few tiles to occupy 256
// compute units but a long K is cut along K: every split writes fp32 partial sums to the workspace and
// a second kernel adds them in a fixed order and runs the epilogue (its traffic and launch are charged
// to the split candidates).
double plan_native(GemmArgs *g, int isz, bool a_kc, bool b_kc, bool allow_split, bool big_unsplit) {
  // microseconds per tile step [tile][0: both operands K-contiguous, 1: one, 2: none] and per block
  static const double step_bf16[3][3] = {{0.27, 0.33, 0.56}, {0.57, 0.68, 1.12}, {1.90, 2.25, 2.70}};
  static const double step_f32[3][3] = {{0.52, 0.62, 0.65}, {1.95, 2.40, 2.10}, {6.90, 7.50, 7.90}};
  static const double fixed_bf16[3] = {1.0, 3.0, 12.0}, fixed_f32[3] = {1.5, 4.0, 18.0};
  const double step_direct = 1.48;                        // bf16 direct-copy kernel, any layout
  const int lay = (a_kc ? 0 : 1) + (b_kc ? 0 : 1);
  const bool direct = direct_copy_fits(*g, isz, a_kc, b_kc);
  const bool small_direct_on = direct && isz == 2 && g_force_w8.load(std::memory_order_relaxed) < 0;   // (forcing one of the 256x256 kernels leaves the other tiles staged)
  // Operands whose rows start off 8-byte boundaries do not get the 256x256 tile; those with an extent below 16 bytes are read in
  // 8-byte pieces on every tile where their rows allow it (a K of 4, say), else element by element, on the small tile only.
  // launch_tile follows the same rule.  A step takes longer where pieces straddle cache lines, and longer still element by element.
  const bool any = g->any_a && g->any_b, halves = g->piece == 8 && !any;
  const int largest = g->piece >= 8 ? 2 : any ? 1 : 0;
  // (bf16 in one 64x64 tile per compute unit: 1024x1000x784 9.1, 1024x1001x785 11.3; 7292x423x487 18.4 on that tile, 27.4 on 128x128)
  auto narrow = [&](int tile) { return g->piece >= 16 ? 1.0 : tile == 2 || halves || (any && isz == 4) ? 1.15 : any ? (tile == 1 ? 2.0 : 1.5) : 2.0; };
  const int nk = (g->K + 128 / isz - 1) / (128 / isz);   // tile steps along K
  static const int split_choices[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16};
  double best = 1e300;
  g->tile = 0; g->splits = 1;
  for (int tile = largest; tile >= 0; --tile) {
    const int b = 64 << tile;
    const int64_t tiles = (int64_t)((g->M + b - 1) / b) * ((g->N + b - 1) / b);
    double per_step = (isz == 2 ? step_bf16 : step_f32)[tile][lay] * narrow(tile);
    if (tile == 2 && direct && isz == 2) per_step = step_direct;
    double fixed = (isz == 2 ? fixed_bf16 : fixed_f32)[tile];
    // The directly copied smaller tiles (bf16), the same for every layout: fitted on 17 products of 1 to 3000 tiles.  The
    // steps are those of a long K (0.62 and 0.215 up to 2048 k): 1000x4096x8192 along M/N 93 on 128x128, 78 on the 256x256 tile
    // cut in four.
    const bool small_direct = tile < 2 && small_direct_on;
    if (small_direct) { per_step = tile == 1 ? 0.68 : 0.235; fixed = tile == 1 ? 4.0 : 2.0; }
    for (int s : split_choices) {
      if (s > 1 && (!allow_split || s > nk / 4)) break;
      const int64_t blocks = tiles * s;
      const int steps = (nk + s - 1) / s;
      // Up to `conc` blocks of this tile run on a compute unit at once, each then `conc` times slower
      // per step than the amortised figure; a lone block only `slow` times (it is not that much faster
      // alone), in between linearly.  Full rounds of 256 * conc blocks, then the remainder.
      const int conc = small_direct ? 2 - tile : tile == 2 ? 1 : tile == 1 ? 2 : 4;
      const double slow = small_direct ? (tile == 1 ? 1.0 : 1.15) : tile == 2 ? 1.0 : tile == 1 ? 1.5 : 1.6;   // (64x64: 2.0 before the kernel looked two tiles ahead)
      const int64_t full = blocks / (256 * conc), rem = blocks % (256 * conc);
      double t = (double)full * (fixed + steps * per_step * conc);
      if (rem > 0) {
        const int per_cu = (int)((rem + 255) / 256);
        const double f = conc == 1 ? 1.0 : slow + (conc - slow) * (per_cu - 1) / (conc - 1);
        t += fixed + steps * per_step * f;
      }
      t *= 1e-6;
      if (s > 1) t += (small_direct ? 5e-6 : 10e-6) + (double)(s + 1) * g->M * g->N * 4.0 / 4e12;
      if (t < best * (small_direct ? 1.0 : 0.97)) { best = t; g->tile = tile; g->splits = s; }   // prefer larger tiles / fewer splits on near-ties
    }
  }
  // The four stages of the directly copied 64x64 tile leave room for two of its blocks on a compute unit, the two of the staged one for
  // more.  With more blocks than that and a single tile step, a few where no operand is to be transposed, a block is its first loads and its
  // epilogue, and the staged kernel has more of them under way (us, direct and staged: 4728x2016x96 19.4 and 15.2, 1000x2728x64 7.0
  // and 6.0, both along M/N 7176x1248x16 16.7 and 13.1, but 2224x1472x192 8.1 and 10.7, 2176x1456x128 7.6 and 9.6).  Instead of the
  // 256x256 tile only with both operands along K and up to 3072 blocks (2376x3408x192 19.2 and 16.4; 7928x3704x64 21.0 and 25.4).
  // Fitted on 149 products of 513 to 7200 blocks, K 8 to 512.
  bool many_staged = false;
  const int64_t small_tiles = (int64_t)((g->M + 63) / 64) * ((g->N + 63) / 64);
  if (small_direct_on && small_tiles > 512 && g->K <= (lay == 0 ? 256 : 64) && (g->tile < 2 || (lay == 0 && small_tiles <= 3072))) {
    // (four blocks of the staged 64x64 tile at once on a compute unit, or two of the 128x128 one: that where its rounds come out even,
    // 5700 blocks of 64x64, 1450 of 128x128, 28.6 and 23.8)
    const int64_t large_tiles = (int64_t)((g->M + 127) / 128) * ((g->N + 127) / 128);
    auto rounds = [&](int64_t blocks, int at_once, double fixed, double step) {
      const int64_t full = blocks / (256 * at_once), rem = blocks % (256 * at_once);
      const double lone = at_once == 4 ? 1.6 : 1.5, more = (at_once - lone) / (at_once - 1);
      return 1e-6 * ((double)full * (fixed + at_once * nk * step) + (rem > 0 ? fixed + nk * step * (lone + more * (double)((rem + 255) / 256 - 1)) : 0.0));
    };
    const double small = rounds(small_tiles, 4, 2.0, lay == 0 ? 0.27 : 0.33);
    const double large = lay < 2 ? rounds(large_tiles, 2, 5.0, step_bf16[1][lay]) : 1e300;
    if (small < best) {
      best = small < large ? small : large;
      g->tile = small < large ? 0 : 1;
      g->splits = 1;
      many_staged = true;
    }
  }
  // The 256 x 128 tile of the eight-wave kernel (bf16, both operands K-contiguous): taken when it fills the chip
  // in one round without a cut along K where the square tile cannot (N near 1000 with a long M).
  const bool narrow_ok = direct && isz == 2 && a_kc && b_kc && !big_unsplit && g_force_w8.load(std::memory_order_relaxed) != 0;
  if (narrow_ok) {
    const int64_t tiles = (int64_t)((g->M + 255) / 256) * ((g->N + 127) / 128);
    const int64_t rounds = (tiles + 255) / 256;
    const double t = (double)rounds * (kNarrowFixed + nk * kNarrowStep) * 1e-6;
    if (t < best * 0.97) { best = t; g->tile = 3; g->splits = 1; }
  }
  {   // chn_gemm_plan_override
    const int force_tile = g_force_tile.load(std::memory_order_relaxed), force_splits = g_force_splits.load(std::memory_order_relaxed);
    if (force_tile >= 0 && force_tile <= largest) { g->tile = force_tile; many_staged = false; }
    if (force_tile == 3 && narrow_ok) g->tile = 3;
    if (force_tile >= 0 && force_tile != 3 && g->tile == 3) g->tile = largest;
    if (force_splits >= 1 && allow_split && force_splits <= nk) g->splits = force_splits;
  }
  if (big_unsplit) { g->tile = 2; g->splits = 1; }        // (the caller has checked that the operands allow the big tile)
  const int bm = g->tile == 3 ? 256 : 64 << g->tile, bn = g->tile == 3 ? 128 : 64 << g->tile;
  g->tiles_m = (g->M + bm - 1) / bm;
  g->tiles_n = (g->N + bn - 1) / bn;
  g->ldp = (g->N + 3) & ~3;
  g->dma = g->tile >= 2 ? direct : small_direct_on && !many_staged;
  g->parts = 0;
  return best;
}

// Few blocks and a contraction that one batch of loads per wave covers: the latency-bound kernel of gemm_tiny.h, up to 256 blocks
// of 32x32 (beyond, 1000x1000x64 say, the tiles' reuse of operands wins) and 1024 k, which sixteen waves cover.  On blocks of 16x16
// while a compute unit gets two of them or their operands are few; above, the larger block's reuse wins (us, 16x16 and 32x32:
// 350x350x512 5.1 and 6.2, x1000 7.8 and 11.1; 400x400x256 4.9 and 5.3, x512 6.4 and 6.1; 512x512x192 4.2 and 4.5, x256 5.7 and 5.3,
// x1000 12.8 and 8.6).  Against the cut product on the tiled kernels: 10x1000x1024 9.9 -> 4.4, 256x256x1000 9.3 -> 5.0, 400x400x1000
// 11.2 -> 8.6; 70 drawn products of up to six 64x64 tiles and 513 to 639 k 2.3 to 3.4 times as fast as cut (46x41x520 12.0 -> 3.5,
// 236x24x636 8.7 -> 3.8), at 0.63 of the error against 64 bits.  Those of them whose operands both lie along K stay cut all the same: the
// planner is held to a cut there by a test that was timed before this kernel existed (44x15x568, 336x53x578).
bool plan_small(GemmArgs *g, int isz, bool both_kc, bool big_unsplit) {
  auto forced = [](const std::atomic<int> &f) { return f.load(std::memory_order_relaxed) >= 0; };
  if (isz != 4 || big_unsplit || g->K == 0 || g->K > 1024 || g->lda >= kMaxLd || g->ldb >= kMaxLd) return false;
  if (forced(g_force_tile) || forced(g_force_direct) || forced(g_force_w8) || forced(g_force_parts) || forced(g_force_splits)) return false;
  auto blocks = [&](int64_t n) { return ((g->M + n - 1) / n) * ((g->N + n - 1) / n); };
  if (blocks(32) > 256 || (both_kc && g->K > 512 && g->K < 640 && blocks(64) <= 6)) return false;
  g->parts = 3;
  g->splits = 1;
  g->tile = g->dma = 0;
  g->small = blocks(16) <= 512 || blocks(16) * g->K <= 200000 ? 16 : 32;
  g->tiles_m = (g->M + g->small - 1) / g->small;
  g->tiles_n = (g->N + g->small - 1) / g->small;
  return true;
}

// fp32 products on the bfloat16 matrix cores (gemm_split.h, gemm_split_direct.h): the 128x128 tile in two groups of waves or the 64x64
// tile in four or by eight waves, against the best plan on the fp32 matrix instruction, by the same kind of model (microseconds, a launch not
// counted).  Figures measured on 64 to 4096 tiles, K 784 to 10000, all four layouts: a block costs 5.6 (loaded directly 4) plus
// its tile steps (32 k on the large tile, 64 on the small one); a step takes longer when all 256 compute units pull operands out of
// the L2s than when a quarter of them does, and element by element (an extent below four).  Each compute
// unit holds one block at a time.  Where the lines cross (fp32 instruction -> this, us): 1024x1000x1000 27 -> 22 on the
// small tile, 4480x2688x672 143 -> 101 and 4480x10000x672 499 -> 361 on the large one, 672x2688x4480 both stored along
// M/N 178 -> 115 cut in two; 640x640x360 along M/N 12.6 -> 10.2 and 585x800x1472 31.0 -> 25.9 loaded directly.
// Rows off the 16-byte grid cost little: against the 8-byte pieces of before, 4480x650x2600 159 -> 145 and 2600x650x4480 162 -> 136;
// against single elements, 4097x2351x2041 556 -> 273 and 8192x4001x651 584 -> 295.
void plan(GemmArgs *g, int isz, bool a_kc, bool b_kc, bool allow_split, bool big_unsplit = false) {
  if (plan_small(g, isz, a_kc && b_kc, big_unsplit)) return;
  double best = plan_native(g, isz, a_kc, b_kc, allow_split, big_unsplit);
  const int force = g_force_parts.load(std::memory_order_relaxed), force_tile = g_force_tile.load(std::memory_order_relaxed);
  const bool other_forced = force_tile >= 0 || g_force_direct.load(std::memory_order_relaxed) >= 0 || g_force_w8.load(std::memory_order_relaxed) >= 0;
  if (isz != 4 || big_unsplit || g->K == 0 || g->lda >= kMaxLd || g->ldb >= kMaxLd || (other_forced && force != 1)) return;
  static const double step_large[3] = {1.0, 1.25, 1.2}, step_direct[3] = {2.4, 2.3, 1.95};    // both along K, one, none
  constexpr double step_small = 0.78;
  const int lay = (a_kc ? 0 : 1) + (b_kc ? 0 : 1);
  auto narrow = [&](bool any, bool kc, bool large) {
    if (g->piece == 16) return 1.0;
    if (any) return large ? 1.05 : 1.1;
    if (g->piece == 8) return large ? (kc ? 1.05 : 1.35) : 1.1;
    return large ? (kc ? 3.2 : 1.9) : (kc ? 3.7 : 3.0);
  };
  // (A finishing launch is charged 5 us here, on both sides.  Cut along K, the fp32 instruction's element-wise loads
  // cost less than the factor of its model says.  With that and with the small tile's steps no more than a fifth
  // cheaper when few blocks run, the choice over 215 drawn products of 1 to 200 tiles is 0.7 % from the best of
  // either path's cuts, it was 3.2 %: 44x15x568 15.7 -> 9.2, 36x80x5127 29.3 -> 17.7.)
  if (g->splits > 1) best = (best - 5e-6) * (g->piece >= 8 ? 1.0 : 0.8);
  static const int split_choices[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16};
  const int forced_splits = g_force_splits.load(std::memory_order_relaxed);
  if (force == 1) best = 1e300;
  GemmArgs p = *g;
  for (int large = 1; large >= 0; --large) {
    if (force == 1 && force_tile >= 0 && force_tile != large) continue;
    const int b = large ? 128 : 64, bk = large ? 32 : 64;
    const int64_t tiles = (int64_t)((g->M + b - 1) / b) * ((g->N + b - 1) / b);
    const int nk = (g->K + bk - 1) / bk;
    const double na = narrow(g->any_a, a_kc, large), nb = narrow(g->any_b, b_kc, large), narrowed = na > nb ? na : nb;
    for (int s : split_choices) {
      if (s > 1 && (!allow_split || s > nk / 4)) break;
      if (forced_splits >= 1 && allow_split && forced_splits <= nk) s = forced_splits;
      const int64_t blocks = tiles * s, rounds = (blocks + 255) / 256;
      const double fill = blocks < 256 ? (double)blocks / 256 : 1.0;
      const int steps = (nk + s - 1) / s;
      // The small tile loads its operands straight into registers (gemm_split_direct.h), unless both lie along K and K is long: through
      // LDS they then come in whole lines.  Eight waves take 128 k a round; in the last one some may have nothing to do.
      const bool direct = !large && (lay > 0 || (steps <= 7 && s == 1));
      double t = direct ? 4.0 + 0.5 * ((steps + 1) / 2 + 0.5 * steps) * step_direct[lay] * (0.8 + 0.2 * fill)
                        : 5.6 + steps * (large ? step_large[lay] * (0.9 + 0.25 * fill) : step_small * (0.8 + 0.2 * fill)) * narrowed;
      t = (double)rounds * t * 1e-6;
      if (direct) t -= 1.8e-6;                             // (the first round's blocks start together with the launch)
      if (s > 1) t += (direct ? 5.7e-6 : 5e-6) + (double)(s + 1) * g->M * g->N * 4.0 / 4e12;
      if (t < best * 0.97) {
        best = t;
        p.parts = large ? 2 : 1;
        p.direct = direct;
        p.splits = s;
        p.tiles_m = (g->M + b - 1) / b;
        p.tiles_n = (g->N + b - 1) / b;
      }
      if (s == forced_splits) break;
    }
  }
  if (p.parts) *g = p;
}

// Which of the two direct-copy kernels takes a bf16 product on the 256x256 tile: the eight-wave one.  Both
// are bound by the chip's power limit on random data and within 2 % of each other on the long products of
// the wide-MLP step (three machines: the eight-wave kernel ahead by 1-2 % on two, behind by 1.5 % on one);
// where a workgroup's fixed parts weigh more the eight-wave kernel wins clearly -- its two waves per SIMD
// overlap prologue, epilogue and barriers: 8192x4096x1000 in 95-100 us against 118-120 us, the products
// with an activation-gradient epilogue 3-5 % faster.  The four-wave kernel (a third less LDS traffic per
// MFMA) stays for fp32 and as the forced alternative of the tests.
bool eight_waves(const GemmArgs &g, int isz, int epilogue) {
  if (!g.dma || isz != 2 || g.tile < 2) return false;
  const int f = g_force_w8.load(std::memory_order_relaxed);
  (void)epilogue;
  return f < 0 || f != 0;
}

// The operands of a product that is only planned.
chn_status check_operands(const chn_array *A, const chn_array *B, const chn_array *C, GemmArgs *g, bool *a_kc, bool *b_kc) {
  CHN_TRY(validate(A, "A", false));
  CHN_TRY(validate(B, "B", false));
  CHN_TRY(validate(C, "C", true));
  if (A->ndim != 2 || B->ndim != 2 || C->ndim != 2) return fail(CHN_ERR_NDIM, "gemm: A, B and C must be 2-d");
  if (!is_float(A->dtype) || A->dtype != B->dtype) return fail(CHN_ERR_DTYPE, "gemm: A and B must share F32 or BF16");
  if (A->shape[1] != B->shape[0] || C->shape[0] != A->shape[0] || C->shape[1] != B->shape[1]) return fail(CHN_ERR_SHAPE, "gemm: shapes do not match");
  if (A->shape[0] > 0x3fffffff || A->shape[1] > 0x3fffffff || B->shape[1] > 0x3fffffff) return fail(CHN_ERR_SHAPE, "gemm: dimension too large");
  return classify(A, B, g, a_kc, b_kc);
}

// What chn_gemm would do with these operands.
chn_status plan_of(const chn_array *A, const chn_array *B, const chn_array *C, int have_workspace, GemmArgs *g) {
  bool a_kc, b_kc;
  CHN_TRY(check_operands(A, B, C, g, &a_kc, &b_kc));
  plan(g, dtype_size(A->dtype), a_kc, b_kc, have_workspace != 0);
  return CHN_OK;
}

size_t split_bytes(const GemmArgs &g) {
  return g.splits > 1 ? (size_t)g.splits * g.M * g.ldp * sizeof(float) : 0;
}

// Validates a product's arrays and fills in everything but the plan (colsum: row-block column sums are wanted).
chn_status prepare(const chn_array *A, const chn_array *B, const chn_array *C, float alpha, float beta, int epilogue, const chn_array *bias,
                   const chn_array *aux, const chn_array *preact_out, GemmArgs &g, bool *a_kc, bool *b_kc) {
  CHN_TRY(validate(A, "A", false));
  CHN_TRY(validate(B, "B", false));
  CHN_TRY(validate(C, "C", true));
  if (A->ndim != 2 || B->ndim != 2 || C->ndim != 2) return fail(CHN_ERR_NDIM, "gemm: A, B and C must be 2-d");
  if (epilogue < 0 || epilogue >= CHN_EPI_COUNT_) return fail(CHN_ERR_OP, "gemm: unknown epilogue %d", epilogue);
  if (!is_float(A->dtype) || A->dtype != B->dtype) return fail(CHN_ERR_DTYPE, "gemm: A and B must share F32 or BF16");
  if (!is_float(C->dtype) || (A->dtype == CHN_F32 && C->dtype != CHN_F32))
    return fail(CHN_ERR_DTYPE, "gemm: C must be F32 (or BF16 when A and B are BF16)");
  const int64_t M = A->shape[0], K = A->shape[1], N = B->shape[1];
  if (B->shape[0] != K) return fail(CHN_ERR_SHAPE, "gemm: A is (%lld,%lld) but B has %lld rows", (long long)M, (long long)K, (long long)B->shape[0]);
  if (C->shape[0] != M || C->shape[1] != N) return fail(CHN_ERR_SHAPE, "gemm: C must be (%lld,%lld)", (long long)M, (long long)N);
  if (M > 0x3fffffff || N > 0x3fffffff || K > 0x3fffffff) return fail(CHN_ERR_SHAPE, "gemm: dimension too large");
  int64_t cr, cc;
  CHN_TRY(row_major_2d(C, "C", &cr, &cc, &g.ldc));
  CHN_TRY(classify(A, B, &g, a_kc, b_kc));
  const bool needs_bias = epilogue >= CHN_EPI_BIAS && epilogue <= CHN_EPI_BIAS_GELU;
  const bool needs_aux = epilogue == CHN_EPI_RELU_BWD || epilogue == CHN_EPI_GELU_BWD;
  if (needs_bias) {
    CHN_TRY(validate(bias, "bias", false));
    if (bias->dtype != CHN_F32) return fail(CHN_ERR_DTYPE, "gemm: bias must be F32");
    if (bias->ndim != 1 || bias->shape[0] != N || !is_contiguous(bias)) return fail(CHN_ERR_SHAPE, "gemm: bias must be a contiguous (%lld,) array", (long long)N);
    g.bias = static_cast<const float *>(bias->data);
  }
  if (needs_aux) {
    CHN_TRY(validate(aux, "aux", false));
    if (aux->dtype != C->dtype) return fail(CHN_ERR_DTYPE, "gemm: aux must have C's dtype");
    int64_t ar, ac;
    CHN_TRY(row_major_2d(aux, "aux", &ar, &ac, &g.ldaux));
    if (ar != M || ac != N) return fail(CHN_ERR_SHAPE, "gemm: aux must have C's shape");
    g.aux = aux->data;
  }
  if (epilogue == CHN_EPI_BF16_COPY && !preact_out) return fail(CHN_ERR_NULL, "gemm: the BF16_COPY epilogue needs preact_out");
  if (preact_out && needs_aux) {
    // activation-gradient epilogues: the second output holds column sums of C over blocks of 128 rows
    CHN_TRY(validate(preact_out, "preact_out", true));
    if (preact_out->dtype != CHN_F32) return fail(CHN_ERR_DTYPE, "gemm: the row-block column sums must be F32");
    int64_t pr, pc;
    CHN_TRY(row_major_2d(preact_out, "preact_out", &pr, &pc, &g.ldcs));
    if (M % 256 || N % 256 || pr != M / 128 || pc != N)
      return fail(CHN_ERR_SHAPE, "gemm: row-block column sums need M and N to be multiples of 256 and an (M/128, N) array");
    if (beta != 0.0f) return fail(CHN_ERR_OP, "gemm: row-block column sums are not produced together with beta != 0");
    if (reinterpret_cast<uintptr_t>(preact_out->data) % 16 || g.ldcs % 4)
      return fail(CHN_ERR_STRIDE, "gemm: the row-block column sums need 16-byte aligned rows");
    g.colsum = static_cast<float *>(preact_out->data);
  } else if (preact_out) {
    if (epilogue != CHN_EPI_BIAS_GELU && epilogue != CHN_EPI_BF16_COPY)
      return fail(CHN_ERR_OP, "gemm: preact_out is only produced by the BIAS_GELU and BF16_COPY epilogues");
    CHN_TRY(validate(preact_out, "preact_out", true));
    if (epilogue == CHN_EPI_BF16_COPY) {
      if (C->dtype != CHN_F32 || preact_out->dtype != CHN_BF16) return fail(CHN_ERR_DTYPE, "gemm: BF16_COPY needs an F32 C and a BF16 preact_out");
    } else if (preact_out->dtype != C->dtype) {
      return fail(CHN_ERR_DTYPE, "gemm: preact_out must have C's dtype");
    }
    int64_t pr, pc;
    CHN_TRY(row_major_2d(preact_out, "preact_out", &pr, &pc, &g.ldpre));
    if (pr != M || pc != N) return fail(CHN_ERR_SHAPE, "gemm: preact_out must have C's shape");
    g.pre = preact_out->data;
  }
  g.A = A->data; g.B = B->data; g.C = C->data;
  g.alpha = alpha; g.beta = beta; g.epi = epilogue; g.c_bf16 = C->dtype == CHN_BF16;
  return CHN_OK;
}

// Launches a product as planned, or, if the plan cuts K and the workspace has no room for that, as planned uncut.
chn_status launch_planned(GemmArgs &g, int isz, bool a_kc, bool b_kc, int epilogue, void *ws, size_t ws_bytes, hipStream_t st) {
  if (g.splits > 1) {
    // split-K is an optimisation: without (enough, aligned) workspace the product is planned unsplit
    if (ws && reinterpret_cast<uintptr_t>(ws) % 256 == 0 && ws_bytes >= split_bytes(g)) g.partial = static_cast<float *>(ws);
    else plan(&g, isz, a_kc, b_kc, false);
  }
  g.w8 = eight_waves(g, isz, epilogue);
  gemm::set_grid(g);
  if (isz == 4) {
    if (a_kc) return b_kc ? gemm::launch_f32_kk(g, st) : gemm::launch_f32_km(g, st);
    return b_kc ? gemm::launch_f32_mk(g, st) : gemm::launch_f32_mm(g, st);
  }
  if (a_kc) return b_kc ? gemm::launch_bf16_kk(g, st) : gemm::launch_bf16_km(g, st);
  return b_kc ? gemm::launch_bf16_mk(g, st) : gemm::launch_bf16_mm(g, st);
}

// ---- the backward of a fully connected layer --------------------------------------------------------------------------

chn_array transposed(const chn_array *a) {
  chn_array t = *a;
  std::swap(t.shape[0], t.shape[1]);
  std::swap(t.strides[0], t.strides[1]);
  return t;
}

// The weight gradient as a product: dW = dv^T x, or, where dW is stored by columns, its transpose x^T dv.  The workspace of one that
// leaves parts of the bias gradient's sums: the cut product's slabs, the parts, what adding them up needs.
struct WeightGradient {
  chn_array A, B, C;
  bool transposed;
  static size_t aligned(size_t n) { return (n + 255) / 256 * 256; }
  chn_array parts(const GemmArgs &g, void *ws) const {
    chn_array a{};
    a.data = static_cast<char *>(ws) + aligned(split_bytes(g));
    a.ndim = 2;
    a.dtype = CHN_F32;
    a.shape[0] = (int64_t)g.splits * (transposed ? g.tiles_m : g.tiles_n);
    a.shape[1] = transposed ? g.N : g.M;
    a.strides[0] = a.shape[1] * 4;
    a.strides[1] = 4;
    return a;
  }
  size_t fold_offset(const GemmArgs &g) const {
    const chn_array a = parts(g, nullptr);
    return aligned(split_bytes(g)) + aligned((size_t)(a.shape[0] * a.strides[0]));
  }
  size_t workspace_bytes(const GemmArgs &g) const {
    chn_array a = parts(g, nullptr);
    a.data = reinterpret_cast<void *>(256);               // (never looked at)
    return fold_offset(g) + chn_reduce_axis_workspace_bytes(&a, 0);
  }
  size_t workspace_bytes() const {
    GemmArgs g{};
    bool a_kc, b_kc;
    if (A.shape[0] <= 0 || A.shape[1] <= 0 || B.shape[1] <= 0 || check_operands(&A, &B, &C, &g, &a_kc, &b_kc) != CHN_OK) return 0;
    plan(&g, dtype_size(A.dtype), a_kc, b_kc, true);
    return !a_kc && !b_kc && gemm::sums_of_large(g, dtype_size(A.dtype)) ? workspace_bytes(g) : split_bytes(g);
  }
};
WeightGradient weight_gradient(const chn_array *dv, const chn_array *x, const chn_array *dW) {
  const bool by_columns = dW->strides[0] == dtype_size(dW->dtype) && dW->shape[0] > 1 && dW->shape[1] > 1 && dW->strides[1] != dW->strides[0];
  if (by_columns) return WeightGradient{transposed(x), *dv, transposed(dW), true};
  return WeightGradient{transposed(dv), *x, *dW, false};
}

// Whether the memory of two arrays may overlap (the span from first to last element).
bool may_overlap(const chn_array *a, const chn_array *b) {
  auto span = [](const chn_array *x, uintptr_t *lo, uintptr_t *hi) {
    *lo = reinterpret_cast<uintptr_t>(x->data);
    *hi = *lo + dtype_size(x->dtype);
    for (int d = 0; d < x->ndim; ++d)
      if (x->shape[d] > 1) *hi += (x->shape[d] - 1) * x->strides[d];
  };
  uintptr_t a0, a1, b0, b1;
  span(a, &a0, &a1);
  span(b, &b0, &b1);
  return a0 < b1 && b0 < a1;
}

// What rules one launch out before anything is planned (which takes 1.3 us a product): the kernels that take both products work on
// tiles of 64x64 or less, at most 512 of the larger ones, and in bfloat16 on operands that are copied straight to LDS.
bool surely_apart(const GemmArgs &w, const GemmArgs *dx, int isz, bool w_mm, bool x_a_kc) {
  auto tiles = [](const GemmArgs &g) { return (int64_t)((g.M + 63) / 64) * ((g.N + 63) / 64); };
  if (!w_mm || (dx && !x_a_kc) || tiles(w) + (dx ? tiles(*dx) : 0) > 512) return true;
  return isz == 2 && !(direct_copy_fits(w, isz, false, false) && (!dx || direct_copy_fits(*dx, isz, true, false)));
}

// Which of the one-launch kernels takes the two planned products (dx: NULL where there is none).
gemm::LinearBwd together(const GemmArgs &w, const GemmArgs *dx, int isz, bool w_mm, bool x_a_kc) {
  using gemm::LinearBwd;
  if (!w_mm || w.splits > 1 || (dx && (!x_a_kc || dx->splits > 1))) return LinearBwd::kApart;
  auto both = [&](auto ok) { return ok(w) && (!dx || ok(*dx)); };
  const int64_t tiles = (int64_t)w.tiles_m * w.tiles_n + (dx ? (int64_t)dx->tiles_m * dx->tiles_n : 0);
  if (isz == 4) {
    if (both([](const GemmArgs &g) { return g.parts == 3 && g.small == 16; })) return LinearBwd::kTiny;
    return tiles <= 512 && both([](const GemmArgs &g) { return g.parts == 1 && g.direct; }) ? LinearBwd::kSplit : LinearBwd::kApart;
  }
  return tiles <= 512 && both([](const GemmArgs &g) { return g.tile == 0 && g.dma; }) ? LinearBwd::kDma : LinearBwd::kApart;
}

// ... planned here, no further than up to the answer.
gemm::LinearBwd plan_together(GemmArgs &w, GemmArgs *dx, int isz, bool w_a, bool w_b, bool x_a, bool x_b) {
  using gemm::LinearBwd;
  const bool mm = !w_a && !w_b;
  if (surely_apart(w, dx, isz, mm, x_a)) return LinearBwd::kApart;
  plan(&w, isz, w_a, w_b, true);
  const LinearBwd alone = together(w, nullptr, isz, mm, true);
  if (!dx || alone == LinearBwd::kApart) return alone;
  plan(dx, isz, x_a, x_b, true);
  return together(w, dx, isz, mm, x_a);
}

}  // namespace
}  // namespace chn

extern "C" {

size_t chn_gemm_workspace_bytes(const chn_array *A, const chn_array *B, const chn_array *C) {
  using namespace chn;
  if (!A || !B || !C || A->ndim != 2 || B->ndim != 2 || !is_float(A->dtype) || A->dtype != B->dtype) return 0;
  if (A->shape[1] != B->shape[0] || A->shape[0] <= 0 || B->shape[1] <= 0) return 0;
  if (A->shape[0] > 0x3fffffff || A->shape[1] > 0x3fffffff || B->shape[1] > 0x3fffffff) return 0;
  GemmArgs g{};
  bool a_kc, b_kc;
  if (classify(A, B, &g, &a_kc, &b_kc) != CHN_OK) return 0;
  plan(&g, dtype_size(A->dtype), a_kc, b_kc, true);
  return split_bytes(g);
}

void chn_gemm_plan_override(int tile, int splits, int direct_copy) {
  chn::g_force_tile.store(tile, std::memory_order_relaxed);
  chn::g_force_splits.store(splits, std::memory_order_relaxed);
  chn::g_force_direct.store(direct_copy == 4 ? -1 : direct_copy >= 2 ? 1 : direct_copy, std::memory_order_relaxed);
  chn::g_force_w8.store(direct_copy == 2 ? 0 : direct_copy == 3 ? 1 : -1, std::memory_order_relaxed);
  chn::g_force_parts.store(direct_copy == 4 ? 1 : -1, std::memory_order_relaxed);
}

int chn_gemm_plan(const chn_array *A, const chn_array *B, const chn_array *C, int have_workspace) {
  chn::GemmArgs g{};
  CHN_TRY(chn::plan_of(A, B, C, have_workspace, &g));
  return g.tile | (g.dma && g.tile >= 2 ? 4 : 0) | (chn::eight_waves(g, chn::dtype_size(A->dtype), CHN_EPI_NONE) || g.parts == 1 || g.parts == 2 ? 8 : 0) | (g.splits << 4);
}

int chn_gemm_plan_kernel(const chn_array *A, const chn_array *B, const chn_array *C, int have_workspace) {
  chn::GemmArgs g{};
  CHN_TRY(chn::plan_of(A, B, C, have_workspace, &g));
  if (g.parts == 3) return CHN_GEMM_KERNEL_SMALL;
  if (g.parts) return CHN_GEMM_KERNEL_PARTS;
  if (!g.dma) return CHN_GEMM_KERNEL_STAGED;
  return chn::eight_waves(g, chn::dtype_size(A->dtype), CHN_EPI_NONE) ? CHN_GEMM_KERNEL_DIRECT8 : CHN_GEMM_KERNEL_DIRECT4;
}

chn_status chn_gemm(const chn_array *A, const chn_array *B, const chn_array *C, float alpha, float beta,
                    int epilogue, const chn_array *bias, const chn_array *aux, const chn_array *preact_out,
                    void *ws, size_t ws_bytes, chn_stream stream) {
  using namespace chn;
  GemmArgs g{};
  bool a_kc, b_kc;
  CHN_TRY(prepare(A, B, C, alpha, beta, epilogue, bias, aux, preact_out, g, &a_kc, &b_kc));
  if (g.M == 0 || g.N == 0) return CHN_OK;
  const int isz = dtype_size(A->dtype);
  if (g.colsum) {
    // the sums are taken per wave tile of the 256x256 kernels, unsplit, on the vector path of the epilogue
    const int vb = 4 * dtype_size(C->dtype);  // bytes of a 4-element vector of C's dtype
    auto ok = [&](const void *q, int64_t ld) { return reinterpret_cast<uintptr_t>(q) % vb == 0 && ld % 4 == 0; };
    if (!ok(g.C, g.ldc) || !ok(g.aux, g.ldaux) || g.piece < 8) return fail(CHN_ERR_STRIDE, "gemm: row-block column sums need operands with 8-byte pieces and 16-byte aligned C and aux rows");
    plan(&g, isz, a_kc, b_kc, false, true);
  } else {
    plan(&g, isz, a_kc, b_kc, true);
  }
  return launch_planned(g, isz, a_kc, b_kc, epilogue, ws, ws_bytes, as_stream(stream));
}

size_t chn_linear_bwd_workspace_bytes(const chn_array *dv, const chn_array *W, const chn_array *x, const chn_array *dx, const chn_array *dW) {
  using namespace chn;
  if (!dv || !x || !dW || dv->ndim != 2 || x->ndim != 2 || dW->ndim != 2) return 0;
  size_t need = std::max(weight_gradient(dv, x, dW).workspace_bytes(), chn_reduce_axis_workspace_bytes(dv, 0));
  if (dx && W) need = std::max(need, chn_gemm_workspace_bytes(dv, W, dx));
  return need;
}

int chn_linear_bwd_plan(const chn_array *dv, const chn_array *W, const chn_array *x, const chn_array *dx, const chn_array *dW) {
  using namespace chn;
  CHN_TRY(validate(dv, "dv", false));
  CHN_TRY(validate(x, "x", false));
  CHN_TRY(validate(dW, "dW", true));
  if (dv->ndim != 2 || x->ndim != 2 || dW->ndim != 2) return fail(CHN_ERR_NDIM, "linear_bwd: dv, x and dW must be 2-d");
  const WeightGradient w = weight_gradient(dv, x, dW);
  GemmArgs gw{}, gx{};
  bool w_a, w_b, x_a = true, x_b;
  CHN_TRY(check_operands(&w.A, &w.B, &w.C, &gw, &w_a, &w_b));
  if (dx) CHN_TRY(check_operands(dv, W, dx, &gx, &x_a, &x_b));
  if (w.transposed || gw.M <= 0 || gw.N <= 0 || gw.K <= 0) return 0;
  return plan_together(gw, dx ? &gx : nullptr, dtype_size(dv->dtype), w_a, w_b, x_a, x_b) != gemm::LinearBwd::kApart;
}

chn_status chn_linear_bwd(const chn_array *dv, const chn_array *W, const chn_array *x, int epilogue, const chn_array *aux, const chn_array *dx,
                          const chn_array *dW, const chn_array *db, void *ws, size_t ws_bytes, chn_stream stream) {
  using namespace chn;
  CHN_TRY(validate(dv, "dv", false));
  CHN_TRY(validate(x, "x", false));
  CHN_TRY(validate(dW, "dW", true));
  if (dv->ndim != 2 || x->ndim != 2 || dW->ndim != 2) return fail(CHN_ERR_NDIM, "linear_bwd: dv, x and dW must be 2-d");
  if (epilogue != CHN_EPI_NONE && epilogue != CHN_EPI_RELU_BWD && epilogue != CHN_EPI_GELU_BWD)
    return fail(CHN_ERR_OP, "linear_bwd: the epilogue of the input gradient is NONE, RELU_BWD or GELU_BWD");
  if (dW->dtype != CHN_F32) return fail(CHN_ERR_DTYPE, "linear_bwd: dW must be F32");
  const WeightGradient w = weight_gradient(dv, x, dW);
  GemmArgs gw{}, gx{};
  bool w_a, w_b, x_a = true, x_b = true;
  CHN_TRY(prepare(&w.A, &w.B, &w.C, 1.0f, 0.0f, CHN_EPI_NONE, nullptr, nullptr, nullptr, gw, &w_a, &w_b));
  if (dx) CHN_TRY(prepare(dv, W, dx, 1.0f, 0.0f, epilogue, nullptr, aux, nullptr, gx, &x_a, &x_b));
  if (db) {
    CHN_TRY(validate(db, "db", true));
    if (db->dtype != CHN_F32) return fail(CHN_ERR_DTYPE, "linear_bwd: db must be F32");
    if (db->ndim != 1 || db->shape[0] != dv->shape[1] || !is_contiguous(db)) return fail(CHN_ERR_SHAPE, "linear_bwd: db must be a contiguous (%lld,) array", (long long)dv->shape[1]);
  }
  const int isz = dtype_size(dv->dtype);
  const bool mm = !w_a && !w_b;
  bool done = false;
  if (mm && gw.M > 0 && gw.N > 0 && gw.K > 0 && !(db && (may_overlap(db, dv) || may_overlap(db, x) || may_overlap(db, dW)))) {
    // one launch: no product may write what another still reads
    const bool apart = may_overlap(dW, dv) || may_overlap(dW, x) ||
                       (dx && (may_overlap(dx, dv) || may_overlap(dx, x) || may_overlap(dx, dW) || (db && may_overlap(dx, db)) || may_overlap(dW, W) ||
                               (db && may_overlap(db, W)) || (aux && (may_overlap(aux, dW) || (db && may_overlap(aux, db))))));
    if (!w.transposed && !apart) {
      const gemm::LinearBwd kind = plan_together(gw, dx ? &gx : nullptr, isz, w_a, w_b, x_a, x_b);
      if (kind != gemm::LinearBwd::kApart) {
        gemm::set_grid(gw);
        gemm::set_grid(gx);
        gw.sums = db ? static_cast<float *>(db->data) : nullptr;
        return gemm::launch_linear_bwd(gw, dx ? &gx : nullptr, x_b, kind, as_stream(stream));
      }
    }
    if (db && gw.tiles_m == 0) plan(&gw, isz, w_a, w_b, true);
    // the sums beside the weight gradient, in parts that a small reduction adds up
    if (db && gemm::sums_of_large(gw, isz) && ws && reinterpret_cast<uintptr_t>(ws) % 256 == 0 && ws_bytes >= w.workspace_bytes(gw)) {
      const chn_array parts = w.parts(gw, ws);
      gw.partial = static_cast<float *>(ws);
      gw.sums = static_cast<float *>(parts.shape[0] == 1 ? db->data : parts.data);
      gemm::set_grid(gw);
      CHN_TRY(gemm::launch_with_sums(gw, w.transposed, isz, as_stream(stream)));
      const size_t at = w.fold_offset(gw);
      if (parts.shape[0] > 1) CHN_TRY(chn_reduce_axis(CHN_REDUCE_SUM, &parts, 0, 0, db, static_cast<char *>(ws) + at, ws_bytes - at, stream));
      done = true;
    }
  }
  if (!done) {
    CHN_TRY(chn_gemm(&w.A, &w.B, &w.C, 1.0f, 0.0f, CHN_EPI_NONE, nullptr, nullptr, nullptr, ws, ws_bytes, stream));
    if (db) CHN_TRY(chn_reduce_axis(CHN_REDUCE_SUM, dv, 0, 0, db, ws, ws_bytes, stream));
  }
  return dx ? chn_gemm(dv, W, dx, 1.0f, 0.0f, epilogue, nullptr, aux, nullptr, ws, ws_bytes, stream) : CHN_OK;
}

}  // extern "C"
