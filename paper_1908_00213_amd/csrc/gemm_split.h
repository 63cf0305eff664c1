// fp32 products on the bfloat16 matrix cores, at fp32 accuracy.
//
// The scheme is that of G. Henry, P. T. P. Tang and A. Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype
// For Higher-Precision Computations", ARITH 2019.  A float x is the sum of three bfloat16 numbers: h = bf16(x),
// m = bf16(x - h), l = bf16(x - h - m), every difference exact (8 + 8 + 8 significant bits, round to nearest even at each
// step, |m| <= 2^-8 |x|, |l| <= 2^-17 |x|), once x is scaled so that l stays in bfloat16's range (kSplitScale).  A product a b is then
//     ah bh + (ah bm + am bh) + (ah bl + am bm + al bh) + [am bl + al bm + al bl],
// and what stands in brackets, at most 2^-24 |a b| and of random sign, is left out: less than the rounding of the product itself.
// Six products of v_mfma_f32_32x32x16_bf16 (32 cycles for 16 k) replace eight of v_mfma_f32_32x32x2_f32
// (64 cycles for 2 k each): 192 instead of 512 cycles of the matrix pipe for the same part of C, with fewer
// roundings of the fp32 accumulator on the way: the error against 64 bits (2-norm) falls from 5.0e-7 to 0.9e-7 at
// K = 784 and from 9.1e-7 to 2.1e-7 at K = 2600.
//
// Measured (us, fp32 instruction -> here, both operands along K): 1024x1000x1000 27.2 -> 22.0, 4480x2688x672 142.8 -> 101.3,
// 4480x10000x672 499 -> 361, 4096x4096x4096 961 -> 688 (200 TFLOP/s, where the instruction's peak is 157).  What bounds the
// large tile is the vector work of the split beside the matrix work (13 instructions per pair of values staged: scaling
// took it from 667 to 688 at 4096^3) and the chip's power limit (1.8 GHz); the small tile, whose waves read 1 KB of LDS for every
// matrix instruction, LDS: it is left to operands that both lie along a long K (gemm_split_direct.h has the others).
#pragma once
#include "gemm_kernel.h"
#include "split.h"

namespace chn {
namespace gemm {

// One operand tile in LDS: sub-tiles of 32 k, each three planes (h, m, l) of ROWS rows, 32 k of bfloat16 = 64 bytes =
// four 16-byte chunks per row.  Chunk q holds k = 4q .. 4q+3 and 16+4q .. 16+4q+3 of the sub-tile (the sum over k is
// order-free as long as both operands agree; this order lets four lanes fetch 64 contiguous bytes of a row per load).
// Four rows share the 256 bytes of the 64 LDS banks; rows and chunks are XORed with (row / 4) % 4 so that 16 lanes
// touch 16 different 16-byte slots in each access pattern: fragment reads (16 rows, one chunk), row-wise writes
// (4 rows x 4 chunks) and transposing writes (rows 4 apart x 4 chunks).
__device__ __forceinline__ int split_off(int row, int q) {
  const int s = (row >> 2) & 3;
  return (row ^ s) * 64 + ((q ^ s) << 4);
}
template <int ROWS> constexpr int kSplitSub = 3 * ROWS * 64;       // bytes of one operand's sub-tile

// Global memory -> registers -> planes in LDS for one operand tile of ROWS rows and SUBS sub-tiles, T threads.
template <int ROWS, int SUBS, bool KC, int T>
struct SplitLoader {
  // unit stride along K: a thread has NU units of eight k of a row (two 16-byte loads each); along M/N: one unit of
  // R rows of k by four m
  static constexpr int NU = KC ? ROWS * SUBS * 4 / T : 1;
  static constexpr int R = ROWS * SUBS * 8 / T;           // 16-byte loads per thread
  static_assert(R == 2 || R == 4, "the tile is dealt out evenly");
  const char *base;                                       // uniform: the tile's first row (KC) / column (MC) at k = 0
  uint32_t off[NU];                                       // byte offset of the unit's first element
  int lim, K, koff;
  int64_t kstride;                                        // bytes between consecutive k (MC)
  int lds;                                                // where the first unit goes inside a stage
  int sw;                                                 // MC: swizzle of the unit's rows
  int down;                                               // MC, pieces at any address: bytes by which the unit's pieces are read early
  bool cut;                                               // ... and whether the tile reaches past the last row (uniform)
  float scale;                                            // +- kSplitScale

  // negate: the k of the odd wave groups are staged with the other sign
  __device__ __forceinline__ void init(int t, const float *p, int64_t ld, int rows_total, int row0, int K_, bool negate) {
    K = K_;
    kstride = ld * 4;
    if constexpr (KC) {
      const int q = t & 3, row = (t >> 2) % ROWS, sub = t / (4 * ROWS);
      koff = sub * 32 + q * 4;
      base = reinterpret_cast<const char *>(p + (int64_t)row0 * ld);
      // (rows past the end re-read the last one: they only feed rows or columns of C that are not stored)
#pragma unroll
      for (int u = 0; u < NU; ++u) off[u] = (uint32_t)((min(row + u * (T / 4), rows_total - 1 - row0) * ld + koff) * 4);
      lim = K - koff;
      scale = negate && (q & 2) ? -kSplitScale : kSplitScale;
      lds = sub * kSplitSub<ROWS> + split_off(row, q);    // (units T / 4 rows apart: whole periods of the swizzle)
    } else {
      constexpr int PAIRS = 4 / R;                        // units that share a group of four k
      const int pair = t % PAIRS, kg = (t / PAIRS) & 7, mc = (t / (8 * PAIRS)) % (ROWS / 4), sub = t / (2 * PAIRS * ROWS);
      koff = sub * 32 + (kg >> 2) * 16 + (kg & 3) * 4 + pair * 2;
      base = reinterpret_cast<const char *>(p + row0) - 16;
      lim = rows_total - row0 - mc * 4;
      down = lim > 0 && lim < 4 ? (4 - lim) * 4 : 0;
      cut = row0 + ROWS > rows_total;
      off[0] = (uint32_t)((koff * ld + (lim > 0 ? mc * 4 : 0)) * 4 + 16);
      sw = mc & 3;
      scale = negate && (kg & 2) ? -kSplitScale : kSplitScale;
      // (rows 4 mc .. 4 mc + 3 share their swizzle; row 4 mc + e sits (e ^ sw) rows behind the group's start)
      lds = sub * kSplitSub<ROWS> + mc * 256 + (((kg & 3) ^ sw) << 4) + (kg >> 2) * 8 + pair * 4;
    }
  }

  // The loads of the tile step whose first k is k0; what lies past K (the last, ragged step and those requested beyond
  // it) is redirected to zeros.  Along K a step whose k all exist (uniform) needs a scalar address and the thread's
  // constant offsets only.
  template <int PB, bool UNIFORM>
  __device__ __forceinline__ void issue(uint4 (&reg)[R], int k0) const {
    if constexpr (KC) {
      const char *p = base + (int64_t)k0 * 4;
      constexpr bool ANY = PB == kAnyPiece;
      if ((UNIFORM || ANY) && k0 + SUBS * 32 <= K) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const uintptr_t a = reinterpret_cast<uintptr_t>(p + (j & 1) * 64) + off[j >> 1];
          if constexpr (ANY) reg[j] = load_any(a);
          else reg[j] = load_chunk<float, PB>(a, 4);
        }
      } else {                                            // (pieces at any address: the last step goes element by element)
#pragma unroll
        for (int j = 0; j < R; ++j)
          reg[j] = load_chunk<float, ANY ? 4 : PB>(reinterpret_cast<uintptr_t>(p) + off[j >> 1] + (j & 1) * 64, lim - k0 - 16 * (j & 1));
      }
    } else {
      const uintptr_t a = reinterpret_cast<uintptr_t>(base) + off[0];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uintptr_t p = a + (int64_t)(k0 + j) * kstride;
        const int n = k0 + koff + j < K ? lim : 0;
        if constexpr (PB == kAnyPiece) reg[j] = load_any(n > 0 ? p - down : reinterpret_cast<uintptr_t>(&kZeroChunk));
        else reg[j] = load_chunk<float, PB>(p, n);
      }
    }
  }

  // Sums over k of what has been loaded (along M/N), by row: four of them a thread, to which PARTS threads contribute.
  static constexpr int PARTS = 8 * SUBS * (4 / R);
  __device__ __forceinline__ void add_up(const uint4 (&reg)[R], float (&s)[4], bool any) const {
    static_assert(!KC && R == 4, "the large tile, along M/N");
    uint4 v[R];
#pragma unroll
    for (int j = 0; j < R; ++j) v[j] = any && cut ? move_down(reg[j], down) : reg[j];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      s[e] += (__uint_as_float((&v[0].x)[e]) + __uint_as_float((&v[1].x)[e])) + (__uint_as_float((&v[2].x)[e]) + __uint_as_float((&v[3].x)[e]));
  }
  // t: as for init; rows: PARTS x ROWS floats
  __device__ __forceinline__ void put_sums(int t, const float (&s)[4], float *rows) const {
    *reinterpret_cast<float4 *>(rows + (t / (2 * ROWS) * 8 + t % 8) * ROWS + t / 8 % (ROWS / 4) * 4) = make_float4(s[0], s[1], s[2], s[3]);
  }

  // any: the pieces were read at any address
  __device__ __forceinline__ void store(const uint4 (&loaded)[R], char *stage, bool any) {
    uint4 reg[R];
#pragma unroll
    for (int j = 0; j < R; ++j) reg[j] = loaded[j];
    if constexpr (!KC) {
      if (any && cut) {
#pragma unroll
        for (int j = 0; j < R; ++j) reg[j] = move_down(reg[j], down);
      }
    }
    constexpr int PLANE = ROWS * 64;
    if constexpr (KC) {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const uint4 a = reg[2 * u], b = reg[2 * u + 1];
        float f[8] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w),
                      __uint_as_float(b.x), __uint_as_float(b.y), __uint_as_float(b.z), __uint_as_float(b.w)};
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] *= scale;
        uint4 h, m, l;
#pragma unroll
        for (int e = 0; e < 4; ++e) split2(f[2 * e], f[2 * e + 1], (&h.x)[e], (&m.x)[e], (&l.x)[e]);
        char *p = stage + lds + u * (T / 4) * 64;
        *reinterpret_cast<uint4 *>(p) = h;
        *reinterpret_cast<uint4 *>(p + PLANE) = m;
        *reinterpret_cast<uint4 *>(p + 2 * PLANE) = l;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t h[R / 2], m[R / 2], l[R / 2];
#pragma unroll
        for (int j = 0; j < R / 2; ++j) {
          const float x = __uint_as_float((&reg[2 * j].x)[e]) * scale, y = __uint_as_float((&reg[2 * j + 1].x)[e]) * scale;
          split2(x, y, h[j], m[j], l[j]);
        }
        char *p = stage + lds + ((e ^ sw) << 6);
        if constexpr (R == 4) {
          *reinterpret_cast<uint2 *>(p) = make_uint2(h[0], h[1]);
          *reinterpret_cast<uint2 *>(p + PLANE) = make_uint2(m[0], m[1]);
          *reinterpret_cast<uint2 *>(p + 2 * PLANE) = make_uint2(l[0], l[1]);
        } else {
          *reinterpret_cast<uint32_t *>(p) = h[0];
          *reinterpret_cast<uint32_t *>(p + PLANE) = m[0];
          *reinterpret_cast<uint32_t *>(p + 2 * PLANE) = l[0];
        }
      }
    }
  }
};

// Workgroup of 4 KG waves: KG groups of 2 x 2 waves, a wave owns 32 TM x 32 TN of the (64 TM) x (64 TN) tile and every
// KG-th 16 k of the contraction; the groups' sums meet in LDS at the end, in group order.  A tile step is 16 KG k.
// The groups exist because a product this small has one tile per compute unit: KG waves on every SIMD
// instead of one, so that loads, splitting, LDS traffic and matrix work of different waves overlap.  Even groups
// multiply first and then split and store their part of the next tile, odd groups the other way round: the matrix pipe
// and the vector pipe of a SIMD are both busy between two barriers.
// The products with a low part go to an accumulator of their own (they are 2^-8 of the others), so the main sum is
// rounded once per 16 k instead of six times.
// The bfloat16 matrix instruction leaves a tiny error of one sign: summed over 10000 k of a softmax gradient times weights,
// the mean error came to -2.6e-8 of the results' size (fp32 instruction: 4e-10), and where many results are added up while
// their random errors cancel, it shows (the bias gradient of the LSTM layer was off by 1.1e-6, 0.92e-6 on the fp32
// instruction).  So the odd groups multiply -A, for nothing: the sign goes in and out with the scale, their error gets the
// other sign, and the mean is 6e-10 (the bias gradient's error 0.5e-6).
template <int TM, int TN, int KG>
constexpr int kSplitStage = (KG / 2) * (kSplitSub<64 * TM> + kSplitSub<64 * TN>);

// Block `block` of the product, and its share of the sums.  lds: two stages.
template <int TM, int TN, int KG, bool A_KC, bool B_KC, int PBA, int PBB, Sums SUMS>
__device__ __forceinline__ void split_block(const GemmArgs &g, unsigned block, char *lds, int &redo) {
  constexpr int BM = 64 * TM, BN = 64 * TN, BK = 16 * KG, SUBS = KG / 2;
  constexpr int A_BYTES = SUBS * kSplitSub<BM>, STAGE = kSplitStage<TM, TN, KG>;
  constexpr int SETS = TM == 1 ? 2 : 1, NT = 256 * KG;    // (the large tile has no registers for a second set)

  const TilePos tp = tile_pos(g, block);
  const int split = tp.split, m0 = tp.tm * BM, n0 = tp.tn * BN;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int grp = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
  const int r = lane & 31, h = lane >> 5;
  const int nk_all = (g.K + BK - 1) / BK;
  const int per_split = split_steps(g, nk_all);
  const int kt0 = split * per_split;
  const int nk = min(nk_all, kt0 + per_split);

  floatx16 acc[TM][TN], low[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.0f;
  if (threadIdx.x == 0) redo = 0;
  {
    // Operands that lie alike are staged by one half of the threads each, with one loader; a mixed pair is staged
    // by all threads together, so that every wave has the same mixture of work.
    constexpr bool kAlike = A_KC == B_KC;
    static_assert(TM == 2 || (A_KC && B_KC), "other layouts of the small tile: gemm_split_direct.h");
    // (a mixed pair of aligned operands: steps of whole k without checks do not pay, 4480x2688x672 120 -> 123 us)
    using LA = SplitLoader<BM, SUBS, A_KC, kAlike ? NT / 2 : NT>;
    using LB = SplitLoader<BN, SUBS, B_KC, kAlike ? NT / 2 : NT>;
    LA la;
    LB lb;
    const bool do_a = wave < 2 * KG;                      // (uniform over a wave)
    const int t = kAlike ? (int)threadIdx.x & (NT / 2 - 1) : (int)threadIdx.x;
    if constexpr (kAlike) {
      la.init(t, static_cast<const float *>(do_a ? g.A : g.B), do_a ? g.lda : g.ldb, do_a ? g.M : g.N, do_a ? m0 : n0, g.K, do_a);
    } else {
      la.init(t, static_cast<const float *>(g.A), g.lda, g.M, m0, g.K, true);
      lb.init(t, static_cast<const float *>(g.B), g.ldb, g.N, n0, g.K, false);
    }
    // staging registers: with two sets taking turns (SETS) loads run two steps ahead of their use, else one
    uint4 ra[LA::R], ra1[LA::R], rb[LB::R], rb1[LB::R];    // (a thread with one role uses ra, ra1 only)
    // sums: what this thread has staged, by its rows of A (columns of B); `due`: stored tiles until the next one that counts
    constexpr bool kSums = SUMS != Sums::kNone, kSumB = SUMS == Sums::kColumnParts;
    static_assert(SUMS != Sums::kRows && (!kSums || (kAlike && BM == BN)), "parts, of what one loader stages");
    float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    const bool sums = kSums && g.sums, summing = sums && do_a != kSumB;
    const int sharing = kSumB ? g.tiles_m : g.tiles_n, share = kSumB ? tp.tm : tp.tn;
    int due = share;
    auto issue = [&](uint4 (&xa)[LA::R], uint4 (&xb)[LB::R], int kt) __attribute__((always_inline)) {
      if constexpr (!kAlike) { la.template issue<PBA, false>(xa, kt * BK); lb.template issue<PBB, false>(xb, kt * BK); }
      else if (PBA == PBB || do_a) la.template issue<PBA, true>(xa, kt * BK);
      else la.template issue<PBB, true>(xa, kt * BK);
    };
    auto store = [&](const uint4 (&xa)[LA::R], const uint4 (&xb)[LB::R], char *stage, int tile) __attribute__((always_inline)) {
      constexpr bool any_a = PBA == kAnyPiece, any_b = PBB == kAnyPiece;
      if constexpr (kSums) {
        if (due == 0) {                                   // (uniform)
          if (summing && tile < nk) la.add_up(xa, sum, kSumB ? any_b : any_a);
          due = sharing;
        }
        --due;
      }
      if constexpr (!kAlike) { la.store(xa, stage, any_a); lb.store(xb, stage + A_BYTES, any_b); }
      else la.store(xa, stage + (do_a ? 0 : A_BYTES), do_a ? any_a : any_b);
    };
    // this group's 16 k inside a stage: sub-tile grp / 2, k-step grp % 2
    const int off = split_off(r, (grp & 1) * 2 + h);
    const int a_at = (grp >> 1) * kSplitSub<BM> + wm * TM * (32 * 64) + off;
    const int b_at = A_BYTES + (grp >> 1) * kSplitSub<BN> + wn * TN * (32 * 64) + off;
    auto product = [&](floatx16 (&d)[TM][TN], const uint4 (&a)[TM], const uint4 (&b)[TN]) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          d[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b[j]), d[i][j], 0, 0, 0);
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    uint4 a[3][TM], b[3][TN];                             // the fragments of this wave's 16 k: parts h, m, l
    auto read_a = [&](const char *stage, int p) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) a[p][i] = *reinterpret_cast<const uint4 *>(stage + a_at + p * (BM * 64) + i * (32 * 64));
    };
    auto read_b = [&](const char *stage, int p) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < TN; ++j) b[p][j] = *reinterpret_cast<const uint4 *>(stage + b_at + p * (BN * 64) + j * (32 * 64));
    };
    // the first two tiles are fetched together
    issue(ra, rb, kt0);
    issue(ra1, rb1, kt0 + 1);
    store(ra, rb, lds, kt0);
    issue(ra, rb, kt0 + 2);
    store(ra1, rb1, lds + STAGE, kt0 + 1);
    if constexpr (SETS == 2) issue(ra1, rb1, kt0 + 3);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 3; ++p) { read_a(lds, p); read_b(lds, p); }
    // One tile step.  Its fragments are in registers when it starts; behind its barrier the next tile lies in `nxt`
    // and nobody reads `cur` any more.  The parts are used in an order that frees them one after the other: each is
    // replaced by the next tile's as soon as its last product has been issued, the two that are needed longest (both h)
    // while the first product of the next step (m m) does without them.  Meanwhile the tile after the next is split
    // and stored into `cur`, by the odd groups before the products, by the even ones after them.
    auto step = [&](auto set_c, int kt) __attribute__((always_inline)) {
      constexpr int SET = decltype(set_c)::value;
      char *cur = lds + (SET == 0 ? 0 : STAGE);
      const char *nxt = lds + (SET == 0 ? STAGE : 0);
      const bool early = grp & 1;
      auto stage_next = [&]() __attribute__((always_inline)) {
        if constexpr (SETS == 2 && SET == 1) { store(ra1, rb1, cur, kt + 2); issue(ra1, rb1, kt + 4); }
        else { store(ra, rb, cur, kt + 2); issue(ra, rb, kt + SETS + 2); }
      };
      __syncthreads();
      if (early) stage_next();
      product(low, a[1], b[1]);
      product(low, a[1], b[0]);
      read_a(nxt, 1);
      product(low, a[0], b[1]);
      read_b(nxt, 1);
      product(low, a[2], b[0]);
      read_a(nxt, 2);
      product(low, a[0], b[2]);
      read_b(nxt, 2);
      product(acc, a[0], b[0]);
      read_a(nxt, 0);
      read_b(nxt, 0);
      if (!early) stage_next();
    };
    int kt = kt0;
    for (; kt + 1 < nk; kt += 2) {
      step(S0{}, kt);
      step(S1{}, kt + 1);
    }
    if (kt < nk) step(S0{}, kt);
    __syncthreads();
    if constexpr (kSums) {
      if (sums) {                                         // (uniform over the workgroup) the threads that share a row add up in LDS
        float *rows = reinterpret_cast<float *>(lds);     // [part][BM]
        if (summing) la.put_sums(t, sum, rows);
        __syncthreads();
        const int first = kSumB ? n0 : m0, extent = kSumB ? g.N : g.M;
        if ((int)threadIdx.x < BM && first + (int)threadIdx.x < extent) {
          float s = 0.0f;
#pragma unroll
          for (int p = 0; p < LA::PARTS; ++p) s += rows[p * BM + threadIdx.x];
          g.sums[(int64_t)(split * sharing + share) * extent + first + threadIdx.x] = s;
        }
        __syncthreads();
      }
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] += low[i][j];
  // An overflow anywhere on the way (a scaled operand or one of its parts, a product, a sum) leaves an infinity or a NaN in
  // this wave's sum, and so do infinities and NaN among the operands: the tile is then multiplied again below.  Rows and
  // columns beyond C, which may hold whatever follows the operands in memory, do not count.
  const float unscale = (grp & 1 ? -1.0f : 1.0f) / (kSplitScale * kSplitScale);
  float bad = 0.0f;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const bool col = n0 + (wn * TN + j) * 32 + r < g.N;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int rows = col ? g.M - m0 - (wm * TM + i) * 32 - 4 * h : 0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        bad = 8 * (v >> 2) + (v & 3) < rows ? __builtin_fmaf(acc[i][j][v], 0.0f, bad) : bad;
        acc[i][j][v] *= unscale;
      }
    }
  }
  if (bad != 0.0f) redo = 1;                              // (0 or NaN)
  // Parts of the accumulators pass between the groups through LDS: [part][wave of the group][value][lane].
  float *meet = reinterpret_cast<float *>(lds) + (wave & 3) * (TN * 16 * 64) + lane;
  constexpr int PART = 4 * TN * 16 * 64;                  // floats of 32 rows of every wave
  auto put = [&](int part, const floatx16 (&x)[TN]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int v = 0; v < 16; ++v) meet[part * PART + (j * 16 + v) * 64] = x[j][v];
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto get = [&](int part, floatx16 (&x)[TN], bool add) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float y = meet[part * PART + (j * 16 + v) * 64];
        x[j][v] = add ? x[j][v] + y : y;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  static_assert((TM == 2 ? 2 : KG - 1) * PART * 4 <= 2 * STAGE, "the parts fit the stages");
  if constexpr (TM == 2) {                                // each group ends up with one of the tile's two 32-row blocks per wave
    static_assert(KG == 2, "one block per group");
    if (grp == 0) put(0, acc[1]); else put(1, acc[0]);
    __syncthreads();
    if (grp == 0) get(1, acc[0], true); else get(0, acc[1], true);
  } else {                                                // the first group takes everything, in group order
    static_assert(TM == 1, "a part for every group but the first");
    if (grp > 0) put(grp - 1, acc[0]);
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int part = 0; part + 1 < KG; ++part) get(part, acc[0], true);
    }
  }
  if (redo) {
    // Some sum of this tile is not finite, with the scaled operands or at all: the first group multiplies the tile again
    // on the fp32 matrix instruction, without ceremony (BM + BN rows of 128 bytes, loaded, stored, multiplied).
    TileLoader<float, BM, A_KC, PBA> la;
    TileLoader<float, BN, B_KC, PBB> lb;
    la.init(static_cast<const float *>(g.A), g.lda, g.M, m0, g.K);
    lb.init(static_cast<const float *>(g.B), g.ldb, g.N, n0, g.K);
    const int rp = lds_row<float>(r), sw = (r >> 1) & 7;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
#pragma unroll 1
    for (int k0 = kt0 * BK; k0 < nk * BK; k0 += 32) {
      if (grp == 0) { la.issue(k0); lb.issue(k0); }
      __syncthreads();
      if (grp == 0) { la.store(lds, k0); lb.store(lds + BM * 128, k0); }
      __syncthreads();
      if (grp == 0) {
        Frags<TM, TN> f;
#pragma unroll 1
        for (int ks = 0; ks < 4; ++ks) {
          f.read(lds + (wm * TM * 32 + rp) * 128, lds + BM * 128 + (wn * TN * 32 + rp) * 128, ((ks * 2 + h) ^ sw) << 4);
          mma<float, TM, TN>(acc, f);
        }
      }
    }
    __syncthreads();
    if constexpr (TM == 2) {
      if (grp == 0) put(0, acc[1]);
      __syncthreads();
      if (grp == 1) get(0, acc[1], false);
    }
  }
  __syncthreads();                                        // nobody reads the parts any more
  if constexpr (TM == 2) {
    floatx16 own[1][TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) own[0][j] = grp == 0 ? acc[0][j] : acc[1][j];
    // (write_out takes wave / 2 for the wave's 32-row block: 2 grp + wm here, where it is 2 wm + grp of the tile)
    write_out<1, TN>(g, own, lds + wave * kEpiStageBytes<1, TN>, m0 + (wm - grp) * 32, n0, split);
  } else {
    if (grp != 0) return;
    write_out<TM, TN>(g, acc, lds + wave * kEpiStageBytes<TM, TN>, m0, n0, split);
  }
}

template <int TM, int TN, int KG, bool A_KC, bool B_KC, int PBA, int PBB, Sums SUMS = Sums::kNone>
__global__ __launch_bounds__(256 * KG) void gemm_split_kernel(GemmArgs g) {
  extern __shared__ __align__(16) char lds[];
  __shared__ int redo;
  split_block<TM, TN, KG, A_KC, B_KC, PBA, PBB, SUMS>(g, blockIdx.x, lds, redo);
}

template <int TM, int TN, int KG, bool A_KC, bool B_KC, int PBA, int PBB, Sums SUMS = Sums::kNone>
chn_status launch_split_piece(const GemmArgs &g, hipStream_t st) {
  constexpr int LDS = 2 * kSplitStage<TM, TN, KG>;
  static_assert(4 * KG * kEpiStageBytes<1, TN> <= LDS && (64 * TM + 64 * TN) * 128 <= LDS, "the stages are reused by what follows the loop");
  auto kern = gemm_split_kernel<TM, TN, KG, A_KC, B_KC, PBA, PBB, SUMS>;
  static std::atomic<bool> configured{false};  // per instantiation
  CHN_TRY(reserve_lds(configured, reinterpret_cast<const void *>(kern), LDS));
  hipLaunchKernelGGL(kern, dim3((unsigned)(g.tiles_m * g.tiles_n * g.splits)), dim3(256 * KG), LDS, st, g);
  CHN_TRY(check_launch("gemm (split fp32)"));
  if (g.splits > 1) {
    const int64_t n = (int64_t)g.M * (g.ldp / 4);
    hipLaunchKernelGGL(gemm_splitk_finish_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g);
    return check_launch("gemm split-K finish");
  }
  return CHN_OK;
}

template <int TM, int TN, int KG, bool A_KC, bool B_KC>
chn_status launch_split(const GemmArgs &g, hipStream_t st) {
  if (g.piece == 16) return launch_split_piece<TM, TN, KG, A_KC, B_KC, 16, 16>(g, st);
  if (g.any_a && g.any_b) return launch_split_piece<TM, TN, KG, A_KC, B_KC, kAnyPiece, kAnyPiece>(g, st);
  if (g.piece == 8) return launch_split_piece<TM, TN, KG, A_KC, B_KC, 8, 8>(g, st);   // (an extent of two or three)
  if (g.any_b) return launch_split_piece<TM, TN, KG, A_KC, B_KC, 4, kAnyPiece>(g, st);
  if (g.any_a) return launch_split_piece<TM, TN, KG, A_KC, B_KC, kAnyPiece, 4>(g, st);
  return launch_split_piece<TM, TN, KG, A_KC, B_KC, 4, 4>(g, st);
}

}  // namespace gemm
}  // namespace chn
