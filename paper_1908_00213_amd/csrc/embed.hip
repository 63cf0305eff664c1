// chn_embed_fwd / chn_embed_bwd: row gather by integer index (the ndarray layer's array indexing,
// Section "GPU Support by CuPy", as the language-model workload uses it) and its gradient.
//
// Forward: one wave copies one row (bit-exact), in 16-byte chunks at whatever address the row has.
// Backward is written as a gather so that it needs no atomics and no workspace and is bit-reproducible: one block owns
// eight neighbouring table rows, scans the id list (wave ballots give the matches as bit masks), and adds the
// matching rows of dout to the table row they belong to in increasing token order.  Rows nobody referenced are
// written as zeros (or left alone when accumulating).  What bounds it is latency and, where a block has many matches, the
// instructions per match.  So up to 4096 ids are scanned at once (sixteen loads per thread in flight, two barriers; one
// or four loads for short lists), everything that finds the next match is scalar (masks read from a lane's register, the
// row taken from the id by a scalar load), the rows of up to four matches are fetched together, and a thread has
// as many columns as the width needs.  Measured (us; 256 ids per scan and one match at a time -> here): 2136 x 1152 with
// 15664 tokens 60.8 -> 32.5, 5105 x 448 with 3776 13.3 -> 7.8, 3264 x 2 with 25 3.3 -> 2.8, 24 x 12 with 1002 85 -> 60.
#include "common.h"

#include <type_traits>

namespace chn {
namespace {

template <typename T, typename L, bool VEC>
__global__ __launch_bounds__(256) void embed_fwd_kernel(const T *table, int64_t tpitch, int64_t V, const L *ids, int64_t N, int64_t D,
                                                        T *out, int64_t opitch) {
  const int lane = threadIdx.x & 63;
  const int64_t n = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  const int64_t id = (int64_t)ids[n];
  T *dst = out + n * opitch;
  if ((uint64_t)id >= (uint64_t)V) {   // an id outside the table is never used as an offset: its row reads as zeros
    for (int64_t d = lane; d < D; d += 64) dst[d] = T(0);
    return;
  }
  const T *src = table + id * tpitch;
  if constexpr (VEC) {
    constexpr int NV = 16 / sizeof(T);
    // (16-byte accesses at whatever element address the rows have; the last one ends with the row)
    for (int64_t d = lane * NV; d < D; d += 64 * NV) {
      const int64_t e = d + NV <= D ? d : D - NV;
      store16_any(dst + e, load16_any(src + e));
    }
  } else {
    for (int64_t d = lane; d < D; d += 64) dst[d] = src[d];
  }
}

constexpr int kMaxColsPerThread = 4;
constexpr int kRowsPerBlock = 8;     // table rows one block owns: the id list is scanned once for all of them

constexpr int kTogether = 4;         // matching rows fetched together

// S: ids per thread and scan; K: columns per thread
template <typename L, int S, int K>
__global__ __launch_bounds__(256) void embed_bwd_kernel(const L *ids, int64_t N, const float *dout, int64_t dpitch, int64_t D,
                                                        float *dtable, int64_t tpitch, int64_t V, int accumulate) {
  static_assert(4 * S <= 64, "one mask per lane");
  __shared__ unsigned long long masks[64];                 // [round][wave]: 64 ids each, in token order
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t v0 = (int64_t)blockIdx.x * kRowsPerBlock;
  const int64_t col0 = (int64_t)blockIdx.y * (256 * K) + threadIdx.x;
  float acc[kRowsPerBlock][K];
#pragma unroll
  for (int r = 0; r < kRowsPerBlock; ++r)
#pragma unroll
    for (int k = 0; k < K; ++k) acc[r][k] = 0.0f;
  int64_t at[K];                                           // (columns past the last one re-read it and are not stored)
#pragma unroll
  for (int k = 0; k < K; ++k) at[k] = min(col0 + k * 256, D - 1);
  for (int64_t base = 0; base < N; base += 256 * S) {
    const int left = (int)min(N - base, (int64_t)(256 * S));
    L id[S];
#pragma unroll
    for (int u = 0; u < S; ++u) id[u] = ids[base + min(u * 256 + (int)threadIdx.x, left - 1)];
#pragma unroll
    for (int u = 0; u < S; ++u) {
      // (one unsigned comparison: ids below v0, negative ones among them, wrap to large numbers.  v0 is a multiple of
      // eight, so an id of -2^31 wraps to eight at least)
      const auto d = (std::make_unsigned_t<L>)id[u] - (std::make_unsigned_t<L>)v0;
      const bool hit = d < kRowsPerBlock && u * 256 + (int)threadIdx.x < left;
      const unsigned long long m = __ballot(hit);
      if (lane == 0) masks[u * 4 + wave] = m;
    }
    __syncthreads();
    const unsigned long long mine = lane < 4 * S ? masks[lane] : 0;
    // From here on everything that finds the matches is uniform and runs on the scalar unit.
    unsigned long long words = __ballot(mine != 0), mm = 0;  // masks with a match (the same on every wave); bits left of the current one
    int w = 0;
    while (words | mm) {
      int hit[kTogether], n_hits = 0;                       // the next matches in token order (past the last: the first again)
#pragma unroll
      for (int q = 0; q < kTogether; ++q) {
        hit[q] = q > 0 ? hit[0] : 0;
        if (words | mm) {
          if (mm == 0) {
            w = __builtin_ctzll(words);
            words &= words - 1;
            mm = (unsigned int)__builtin_amdgcn_readlane((int)mine, w) |
                 (unsigned long long)(unsigned int)__builtin_amdgcn_readlane((int)(mine >> 32), w) << 32;
          }
          hit[q] = w * 64 + __builtin_ctzll(mm);
          mm &= mm - 1;
          n_hits = q + 1;
        }
      }
      int row_of[kTogether];                                // (the id again, as a scalar)
#pragma unroll
      for (int q = 0; q < kTogether; ++q) row_of[q] = (int)(ids[base + hit[q]] - (L)v0);
      float x[kTogether][K];
#pragma unroll
      for (int q = 0; q < kTogether; ++q) {
        const float *row = dout + (base + hit[q]) * dpitch;
#pragma unroll
        for (int k = 0; k < K; ++k) x[q][k] = row[at[k]];
      }
      __builtin_amdgcn_sched_barrier(0);                    // all loads first
#pragma unroll
      for (int q = 0; q < kTogether; ++q)
        if (q < n_hits) {
#pragma unroll
          for (int r = 0; r < kRowsPerBlock; ++r)
            if (r == row_of[q]) {
              asm("" : "+v"(acc[r][0]));                    // (a branch: eight rows' sums, seven of them dropped, cost more)
#pragma unroll
              for (int k = 0; k < K; ++k) acc[r][k] += x[q][k];
            }
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < kRowsPerBlock; ++r) {
    if (v0 + r >= V) break;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int64_t c = col0 + k * 256;
      if (c < D) {
        float *q = dtable + (v0 + r) * tpitch + c;
        *q = accumulate ? *q + acc[r][k] : acc[r][k];
      }
    }
  }
}

chn_status check_ids(const chn_array *ids, int64_t *N) {
  CHN_TRY(validate(ids, "ids", false));
  if (!is_index(ids->dtype)) return fail(CHN_ERR_DTYPE, "embed: ids must be I32 or I64");
  if (ids->ndim != 1 || !is_contiguous(ids)) return fail(CHN_ERR_SHAPE, "embed: ids must be a contiguous 1-d array");
  *N = ids->shape[0];
  return CHN_OK;
}

}  // namespace
}  // namespace chn

extern "C" {

chn_status chn_embed_fwd(const chn_array *table, const chn_array *ids, const chn_array *out, chn_stream stream) {
  using namespace chn;
  int64_t N, V, D, tp, on, od, op;
  CHN_TRY(check_ids(ids, &N));
  CHN_TRY(validate(table, "table", false));
  CHN_TRY(validate(out, "out", true));
  if (!is_float(table->dtype) || out->dtype != table->dtype) return fail(CHN_ERR_DTYPE, "embed: table and out must share F32 or BF16");
  CHN_TRY(row_major_2d(table, "table", &V, &D, &tp));
  CHN_TRY(row_major_2d(out, "out", &on, &od, &op));
  if (on != N || od != D) return fail(CHN_ERR_SHAPE, "embed: out must have shape (%lld,%lld)", (long long)N, (long long)D);
  if (N == 0 || D == 0) return CHN_OK;
  if (V == 0) return fail(CHN_ERR_SHAPE, "embed: empty table");
  const int isz = dtype_size(table->dtype);
  const bool vec = D * isz >= 16;
  const unsigned blocks = (unsigned)((N + 3) / 4);
  hipStream_t st = as_stream(stream);
  const bool i32 = ids->dtype == CHN_I32;
#define CHN_GO(T, L, V_)                                                                                     \
  hipLaunchKernelGGL((embed_fwd_kernel<T, L, V_>), dim3(blocks), dim3(256), 0, st, static_cast<const T *>(table->data), tp, V, \
                     static_cast<const L *>(ids->data), N, D, static_cast<T *>(out->data), op)
  if (isz == 4) {
    if (i32) { if (vec) CHN_GO(float, int32_t, true); else CHN_GO(float, int32_t, false); }
    else { if (vec) CHN_GO(float, int64_t, true); else CHN_GO(float, int64_t, false); }
  } else {
    if (i32) { if (vec) CHN_GO(bf16_raw, int32_t, true); else CHN_GO(bf16_raw, int32_t, false); }
    else { if (vec) CHN_GO(bf16_raw, int64_t, true); else CHN_GO(bf16_raw, int64_t, false); }
  }
#undef CHN_GO
  return check_launch("embed_fwd");
}

chn_status chn_embed_bwd(const chn_array *ids, const chn_array *dout, const chn_array *dtable,
                         int accumulate, chn_stream stream) {
  using namespace chn;
  int64_t N, V, D, tp, dn, dd, dp;
  CHN_TRY(check_ids(ids, &N));
  CHN_TRY(validate(dout, "dout", false));
  CHN_TRY(validate(dtable, "dtable", true));
  if (dout->dtype != CHN_F32 || dtable->dtype != CHN_F32) return fail(CHN_ERR_DTYPE, "embed: dout and dtable must be F32");
  CHN_TRY(row_major_2d(dtable, "dtable", &V, &D, &tp));
  CHN_TRY(row_major_2d(dout, "dout", &dn, &dd, &dp));
  if (dn != N || dd != D) return fail(CHN_ERR_SHAPE, "embed: dout must have shape (%lld,%lld)", (long long)N, (long long)D);
  if (V == 0 || D == 0) return CHN_OK;
  if (V > 0x7fffffff) return fail(CHN_ERR_SHAPE, "embed: table too large");
  const int cols = (int)min((D + 255) / 256, (int64_t)kMaxColsPerThread);
  dim3 grid((unsigned)((V + kRowsPerBlock - 1) / kRowsPerBlock), (unsigned)((D + 256 * cols - 1) / (256 * cols)));
  if (grid.y > 65535) return fail(CHN_ERR_SHAPE, "embed: rows too wide");
  hipStream_t st = as_stream(stream);
#define CHN_BWD(L, S, K) \
  hipLaunchKernelGGL((embed_bwd_kernel<L, S, K>), grid, dim3(256), 0, st, static_cast<const L *>(ids->data), N, \
                     static_cast<const float *>(dout->data), dp, D, static_cast<float *>(dtable->data), tp, V, accumulate)
#define CHN_BWD_K(L, S) \
  do { if (cols == 1) CHN_BWD(L, S, 1); else if (cols == 2) CHN_BWD(L, S, 2); else if (cols == 3) CHN_BWD(L, S, 3); else CHN_BWD(L, S, 4); } while (0)
#define CHN_BWD_S(L) \
  do { if (N <= 256) CHN_BWD_K(L, 1); else if (N <= 1024) CHN_BWD_K(L, 4); else CHN_BWD_K(L, 16); } while (0)
  if (ids->dtype == CHN_I32) CHN_BWD_S(int32_t);
  else CHN_BWD_S(int64_t);
#undef CHN_BWD_S
#undef CHN_BWD_K
#undef CHN_BWD
  return check_launch("embed_bwd");
}

}  // extern "C"
