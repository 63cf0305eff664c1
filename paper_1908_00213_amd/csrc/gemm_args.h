// Kernel argument block of the GEMM kernels (shared by the host API and the kernel families).
#pragma once
#include <stdint.h>

namespace chn {
namespace gemm {

struct GemmArgs {
  const void *A, *B;
  void *C;
  int M, N, K;
  int64_t lda, ldb, ldc;  // elements; for a K-contiguous operand the stride between rows (m or n),
                          // otherwise the stride between consecutive k
  float alpha, beta;
  int epi;
  int c_bf16;             // C / aux / preact dtype: 0 fp32, 1 bf16
  const float *bias;
  const void *aux;
  int64_t ldaux;
  void *pre;
  int64_t ldpre;
  // what only the host reads, kept short: a launch copies all of this
  int8_t piece;           // bytes per global load piece (16, 8 or the item size), common to A and B
  int8_t piece_a, piece_b;  // what A and B allow each
  int8_t any_a, any_b;    // whether the unit-stride extent of A, of B holds a 16-byte piece (which the smaller tiles read at any address)
  int8_t piece_exact;     // the same when no piece may hang over the end of a row (direct-copy kernels)
  int8_t tile;            // macro tile: 2 = 256x256, 1 = 128x128, 0 = 64x64
  int8_t dma;             // big tile: K-contiguous operands go to LDS by direct global-to-LDS loads
  int8_t w8;              // ... by the kernel that works with eight waves (bf16)
  int8_t parts;           // fp32 on the bfloat16 matrix cores (gemm_split.h): 0 no, 1 on 64x64 tiles, 2 on 128x128 tiles;
                          // 3: the latency-bound kernel for few tiles and a short K (gemm_tiny.h), whose blocks are
  int8_t small;           // 16x16 or 32x32
  int8_t direct;          // parts == 1: operands straight to the registers (gemm_split_direct.h)
  int tiles_m, tiles_n;
  int splits;             // number of K splits (1 = none)
  float *partial;         // split-K: [splits][M][ldp] fp32 partial sums in the caller's workspace
  int64_t ldp;
  float *colsum;          // activation-gradient epilogues, 256x256 tile only: [M / 128][N] column sums of C over
                          // blocks of 128 rows (values as stored), or NULL
  int64_t ldcs;
  // reciprocals (set_grid) by which a block finds its tile: of the tiles, of eight tile rows, of the tile rows behind the last eight, of
  // the tile columns, of the splits
  unsigned per_tiles, per_eight, per_rest, per_column, per_splits;
  float *sums;            // backward of a fully connected layer (linear_bwd.hip): sums over k of A's rows or B's columns, or NULL
};

// At most 2^32 / d and more than that less one: the high word of n times it is n / d or one less, for every n.
constexpr unsigned reciprocal(unsigned d) { return d > 0 ? 0xffffffffu / d : 0; }
inline void set_grid(GemmArgs &g) {
  g.per_tiles = reciprocal((unsigned)g.tiles_m * (unsigned)g.tiles_n);
  g.per_eight = reciprocal(8 * (unsigned)g.tiles_n);
  g.per_rest = reciprocal(g.tiles_m % 8);
  g.per_column = reciprocal(g.tiles_n);
  g.per_splits = reciprocal(g.splits);
}

// Which sums a product's kernel leaves beside C.  kRows: [M], A's rows, by the blocks of the first tile column.  kRowParts,
// kColumnParts: [splits * tiles_n][M] of A's rows, [splits * tiles_m][N] of B's columns: the blocks that stage the same rows of
// A (columns of B) take every tiles_n-th (tiles_m-th) tile step of it each, so that none has more to do than the others.
enum class Sums { kNone, kRows, kRowParts, kColumnParts };

}  // namespace gemm
}  // namespace chn
