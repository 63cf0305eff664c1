// chn_reduce_axis: fold + or max over one axis (Section "Custom CUDA Kernels": the reduction kernel).
//
// The host turns (view, axis) into one of three shapes of work:
//   ROW  the reduced axis has unit stride and the kept dimensions merge into one pitched row index:
//        a group of G lanes (8 / 64 / 256) walks each row with 16-byte loads, folds through wave
//        butterflies (and LDS across the four waves of a block for G = 256);
//   COL  the innermost kept dimension has unit stride: (outer O, reduced R, inner I).  Each thread
//        owns one 16-byte column group, a block is 64 column groups x 4 row lanes, and R is split
//        over S blocks whose fp32 partial sums land in the caller's workspace and are folded by a
//        second launch of the same kernel -- no atomics, so results are bit-reproducible; a short stack
//        of rows that fits the caches (a bias gradient) is folded by one launch of tall, narrow blocks;
//   GEN  anything else: one thread per output element.
// A transposed 2-d view simply swaps ROW and COL.  HBM-bound: the input is read exactly once.
#include "common.h"

#include <algorithm>
#include <mutex>

namespace chn {
namespace {

// Partial sums of chn_reduce_axis_static: one array per GPU for the life of the process.  In host code
// the name is only a handle for hipGetSymbolAddress; kernels receive the address that call returns.
constexpr size_t kScratchBytes = (size_t)CHN_REDUCE_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices] = {nullptr};
std::mutex g_scratch_mutex;

// Address of the current device's copy of `scratch` (looked up once per device, with that device current).
chn_status scratch_of_current_device(void **out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(CHN_ERR_LAUNCH, "reduce (static scratch): hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return fail(CHN_ERR_LAUNCH, "reduce (static scratch): device ordinal %d not supported", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return fail(CHN_ERR_LAUNCH, "reduce (static scratch): hipGetSymbolAddress: %s", hipGetErrorString(e));
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return CHN_OK;
}

template <int OP> __device__ __forceinline__ float fold(float a, float b) {
  if constexpr (OP == CHN_REDUCE_SUM) return a + b; else return fmaxf(a, b);
}
template <int OP> __device__ __forceinline__ float identity() {
  if constexpr (OP == CHN_REDUCE_SUM) return 0.0f; else return -INFINITY;
}
// four bytes of input elements that hold it
template <int OP, typename T> __device__ __forceinline__ uint32_t identity_word() {
  return OP == CHN_REDUCE_SUM ? 0u : sizeof(T) == 2 ? 0xff80ff80u : 0xff800000u;
}

enum { KIND_EMPTY = 0, KIND_ROW = 1, KIND_COL = 2, KIND_GEN = 3 };

struct RPlan {
  int kind = KIND_GEN;
  int64_t len = 0, total_out = 0;
  int64_t sR = 0;            // element stride of the reduced axis
  // kept dimensions after dropping length-1 and merging
  int nk = 0;
  int64_t kshape[CHN_MAX_NDIM] = {0}, kstr[CHN_MAX_NDIM] = {0};
  // COL
  int64_t O = 1, I = 1, sO = 0;
  int split = 1;
  int64_t rows_per_split = 0;
  bool vec = false;
  int tx = 64;               // column groups per block
  size_t ws_bytes = 0;       // COL: partial sums of the slices (required)
  // ROW: a long row that too few blocks would work on is cut in slices whose results a second launch folds, where the
  // caller's workspace has room for them (optional: without it one block folds the slices of a row in turn)
  int slices = 1;
  int64_t slice = 0;
  size_t slice_bytes = 0;
};

// Few long rows (the sum over everything is one): one block moves 16 KB per memory latency, so the sum over 1024 x 1001
// fp32 took 136 us in a single block, 7.8 us cut in slices; the sum over 16 x 16384 37 and 7.9.  Worth it from kCutRow
// elements on, as long as the rows alone do not fill the chip; but the second launch costs a microsecond, so the shortest of
// these stay whole (whatever workspace there is): one row of 32768 bf16 2.9 us against 4.4 in slices, 60000 3.8 and 4.4, 80000
// 4.6 and 4.4; fp32 40000 3.8 and 4.4, 60000 4.6 and 4.4, but 32 rows of 40000 5.5 and 4.9.
constexpr int64_t kCutRow = 32768, kCutRows = 256, kSliceElems = 4096;
constexpr int kMaxSlices = 8192;                            // over all rows
// Many rows of kWaveRowLen elements and more, up to kWaveRowBytes, are a wave's each instead of a block's, eight vectors per lane in
// flight (us, a block's against a wave's: 8192 x 2048 bf16 6.4 and 4.4, 8192 x 4001 bf16 12.2 and 11.2, 8192 x 2500 fp32 13.4 and 11.4).
// Fewer rows leave the chip too few loads in flight (1024 x 4001 bf16 3.2 and 3.4, 2000 x 2500 fp32 3.3 and 3.7; at 3000 it depends on
// the length), and so do longer ones to each wave (16384 x 4096 fp32 38 and 42).
constexpr int64_t kWaveRows = 4096, kWaveRowLen = 2048, kWaveRowBytes = 10240;
bool cut_pays(int64_t rows, int64_t len, int isz) {
  return len >= (isz == 2 ? 65536 : rows <= 8 ? 57344 : rows <= 16 ? 45056 : kCutRow);
}

// COL kernel block shapes (column groups x row lanes = 256 threads): 16 x 16 for the large streaming
// case (more column blocks, hence fewer row splits and a smaller second pass), 64 x 4 otherwise.
constexpr int kColTXWide = 16, kColTXMid = 32, kColTXNarrow = 64;
// A stack of at most kShortRows rows that fits the caches (a bias gradient: the column sums of one
// layer's output gradient) takes a single launch instead: blocks 4 column groups wide and 64 row lanes
// tall, every lane's loads (up to 16) in flight at once, so the launch lasts about one memory latency.
constexpr int kColTXShort = 4;
constexpr int64_t kShortRows = 2048, kShortBytes = 8 << 20;

// alone: not one of several passes that share a workspace (whose size must not grow with this one's partial sums)
chn_status make_rplan(const chn_array *in, int axis, RPlan *p, bool alone) {
  CHN_TRY(validate(in, "in", false));
  if (!is_float(in->dtype)) return fail(CHN_ERR_DTYPE, "reduce: input must be F32 or BF16");
  if (in->ndim < 1) return fail(CHN_ERR_NDIM, "reduce: input needs at least one dimension");
  int ax = axis < 0 ? axis + in->ndim : axis;
  if (ax < 0 || ax >= in->ndim) return fail(CHN_ERR_AXIS, "reduce: axis %d out of range for ndim %d", axis, in->ndim);
  const int isz = dtype_size(in->dtype);
  p->len = in->shape[ax];
  p->sR = p->len > 1 ? in->strides[ax] / isz : 1;
  p->total_out = 1;
  int nk = 0;
  for (int d = 0; d < in->ndim; ++d) {
    if (d == ax) continue;
    p->total_out *= in->shape[d];
    if (in->shape[d] == 1) continue;
    p->kshape[nk] = in->shape[d];
    p->kstr[nk] = in->strides[d] / isz;
    ++nk;
  }
  if (p->total_out == 0 || p->len == 0) { p->kind = KIND_EMPTY; p->nk = nk; return CHN_OK; }
  int w = 0;
  for (int d = 1; d < nk; ++d) {
    if (p->kstr[w] == p->kstr[d] * p->kshape[d]) {
      p->kshape[w] *= p->kshape[d]; p->kstr[w] = p->kstr[d];
    } else {
      ++w; p->kshape[w] = p->kshape[d]; p->kstr[w] = p->kstr[d];
    }
  }
  nk = nk == 0 ? 0 : w + 1;
  p->nk = nk;
  if ((p->sR == 1 || p->len == 1) && nk <= 1) {
    p->kind = KIND_ROW;
    const int64_t rows = nk == 1 ? p->kshape[0] : 1;
    if (rows < kCutRows && p->len >= kCutRow) {
      int64_t s = (p->len + 2 * kSliceElems - 1) / (2 * kSliceElems);
      if (s * rows < 256) s = std::min((p->len + kSliceElems - 1) / kSliceElems, (256 + rows - 1) / rows);   // one block per compute unit
      if (s * rows > kMaxSlices) s = kMaxSlices / rows;                 // (rows < 256: at least 32)
      p->slice = ((p->len + s - 1) / s + 1023) / 1024 * 1024;
      p->slices = (int)((p->len + p->slice - 1) / p->slice);
      p->slice_bytes = (size_t)(rows * p->slices) * sizeof(float);
    }
    return CHN_OK;
  }
  if (nk >= 1 && nk <= 2 && p->kstr[nk - 1] == 1) {
    p->kind = KIND_COL;
    p->I = p->kshape[nk - 1];
    p->O = nk == 2 ? p->kshape[0] : 1;
    p->sO = nk == 2 ? p->kstr[0] : 0;
    const int n = 16 / isz;
    // 16-byte accesses wherever a row holds one; they may start at any element address (10000 x 4001 bf16 column sums
    // 29.8 -> 19.8 us against one element per access, 12000 x 1500 21.3 -> 15.8).  Off the 16-byte grid one element per
    // access stays the better where it gives the more blocks and a short chain per thread: small stacks of rows
    // (376 x 8 bf16 2.5 against 3.7 us, 256 x 1109 3.0 and 4.2) and mid-size widths (9340 x 451 bf16 8.2 and 10.7, 2657 x 179
    // fp32 5.8 and 6.5).
    const bool aligned = reinterpret_cast<uintptr_t>(in->data) % 16 == 0 && p->I % n == 0 && p->sR % n == 0 && p->sO % n == 0;
    const bool stack = p->len <= kShortRows && p->O * p->len * p->I * isz <= kShortBytes / 8 && (isz == 2 || p->len > 128);
    const bool mid = isz == 2 ? p->I > 128 && p->I < 1280 && p->len > kShortRows : p->I > 128 && p->I < 256;
    p->vec = p->I >= n && (aligned || !(stack || mid));
    const int64_t groups = p->vec ? (p->I + n - 1) / n : p->I;
    p->tx = (p->vec && groups >= 512 && p->len >= 1024) ? (isz == 2 && groups >= 1024 ? kColTXMid : kColTXWide) : kColTXNarrow;
    if (p->vec && groups <= 32) p->tx = groups <= 4 && p->len >= 1024 ? kColTXShort : groups <= 16 ? kColTXWide : kColTXMid;   // no idle column lanes (16384 x 16 fp32 14.0 -> 7.8 us)
    if (p->vec && groups >= 64 && p->len <= 64) p->tx = kColTXWide;   // 16 row lanes: one batch of loads per thread
    const int64_t cols_per_block = (int64_t)p->tx * (p->vec ? n : 1);
    const int64_t blocks_xy = ((p->I + cols_per_block - 1) / cols_per_block) * p->O;
    // Measured on 8192 x 8192: many short blocks (8 rows per thread, 16 of bf16) stream best.
    const int rpt = isz == 2 ? 16 : 8;   // rows per thread (bf16: half the partial sums for the second pass, -5 %)
    int64_t s = p->len / (rpt * (256 / p->tx));
    // (few blocks: down to one batch of loads per thread, as long as the second pass stays one batch, too)
    if (blocks_xy * s < 256) s = std::max(s, std::min(std::min(256 / blocks_xy, (int64_t)64), p->len / (4 * (256 / p->tx))));
    if (blocks_xy * s > 16384) s = 16384 / blocks_xy;
    if (p->len <= 64) s = 1;        // a short stack of rows (e.g. per-row-block sums): one launch, a few loads per thread
    // (rows off the 16-byte grid: partial sums of at most 4 MiB, which the built-in scratch of
    // chn_reduce_axis_static holds for every shape)
    const int64_t most = (4 << 20) / (p->O * p->I * (int64_t)sizeof(float) + 1);
    if (!aligned && s > most) s = most;
    if (s < 1) s = 1;
    if (s > 1024) s = 1024;
    if (s > 1 && p->len <= kShortRows && p->O * p->len * p->I * isz <= (p->vec ? kShortBytes : kShortBytes / 8)) {
      p->tx = kColTXShort;
      s = 1;
    }
    p->split = (int)s;
    p->rows_per_split = (p->len + s - 1) / s;
    // whole batches of eight rows per thread (10000 x 4001 bf16, 65 rows a slice -> 64: 22.0 -> 21.0 us), where the partial sums
    // stay within what chn_reduce_axis_static holds
    const int64_t batch = 8 * (256 / p->tx);
    if (alone && p->vec && (isz == 2 || p->tx != kColTXWide) && p->rows_per_split > batch && blocks_xy * s >= 1024) {
      const int64_t down = p->rows_per_split / batch * batch, slices = (p->len + down - 1) / down;
      if (slices <= 1024 && (aligned || slices <= most) && slices * p->O * p->I * (int64_t)sizeof(float) <= (int64_t)kScratchBytes) p->rows_per_split = down;
    }
    p->split = (int)((p->len + p->rows_per_split - 1) / p->rows_per_split);
    p->ws_bytes = p->split > 1 ? (size_t)p->split * p->O * p->I * sizeof(float) : 0;
    return CHN_OK;
  }
  p->kind = KIND_GEN;
  return CHN_OK;
}

// ------------------------------------------------------------------------------------------------
template <typename Tout>
__global__ __launch_bounds__(256) void fill_kernel(Tout *out, int64_t n, float v) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) Elem<Tout>::store(out + i, v);
}

// One lane's share of a row of `len` elements: G lanes, four accumulators each, folded in an order that depends on len
// alone.  BATCHES of four 16-byte loads are in flight at once, and so are those of the last vectors, fewer than a batch, and of
// the elements behind them (one after the other they took a trip to memory each: 10000 x 4001 bf16 16.3 -> 14.5 us, 8192 x 1000 fp32
// 6.1 -> 5.7; a lane without a vector loads none: with the last one in its place 16384 x 500 bf16 takes 6.1, so 4.5).
template <int OP, typename Tin, int G, bool VEC, int BATCHES>
__device__ __forceinline__ float fold_row(const Tin *p, int64_t len, int g) {
  float acc[4] = {identity<OP>(), identity<OP>(), identity<OP>(), identity<OP>()};
  if constexpr (VEC) {
    constexpr int N = Vec16<Tin>::N;
    const int64_t nvec = len / N;
    int64_t v = g;
    auto batches = [&](auto count) __attribute__((always_inline)) {
      constexpr int U = 4 * decltype(count)::value;
      for (; v + (U - 1) * G < nvec; v += U * G) {
        Vec16<Tin> x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = load16_any_nt(p + (v + u * G) * N);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < N; ++i) acc[u & 3] = fold<OP>(acc[u & 3], x[u].get(i));
      }
    };
    if constexpr (BATCHES > 1) batches(std::integral_constant<int, BATCHES>{});
    batches(std::integral_constant<int, 1>{});
    const int left = (int)(nvec - v);
    Vec16<Tin> x[3];
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (u * G < left) x[u] = load16_any(p + (v + u * G) * N);
    const int64_t at = nvec * N + g;
    const float rest = at < len ? Elem<Tin>::load(p + at) : identity<OP>();   // (at most N - 1 of them, G >= N lanes)
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (u * G < left) {
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i & 3] = fold<OP>(acc[i & 3], x[u].get(i));
      }
    acc[1] = fold<OP>(acc[1], rest);
  } else {
    int64_t c = g;
    for (; c + 3 * G < len; c += 4 * G) {
      float x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = Elem<Tin>::load(p + c + u * G);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = fold<OP>(acc[u], x[u]);
    }
    for (; c < len; c += G) acc[0] = fold<OP>(acc[0], Elem<Tin>::load(p + c));
  }
  return fold<OP>(fold<OP>(acc[0], acc[1]), fold<OP>(acc[2], acc[3]));
}
// The same for a mid-size row that one wave folds: eight vectors per lane in flight, in the last, partial batch too.
template <int OP, typename Tin>
__device__ __forceinline__ float fold_row_by_wave(const Tin *p, int64_t len, int g) {
  constexpr int N = Vec16<Tin>::N, G = 64, U = 8;
  float acc[4] = {identity<OP>(), identity<OP>(), identity<OP>(), identity<OP>()};
  const int64_t nvec = len / N, at = nvec * N + g;
  int64_t v = 0;
  for (; v + U * G <= nvec; v += U * G) {
    Vec16<Tin> x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = load16_any_nt(p + (v + g + u * G) * N);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < N; ++i) acc[u & 3] = fold<OP>(acc[u & 3], x[u].get(i));
  }
  const int left = (int)(nvec - v);
  const Tin *q = p + v * N;
  Vec16<Tin> x[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (g + u * G < left) x[u] = load16_any(q + (g + u * G) * N);
  const float rest = at < len ? Elem<Tin>::load(p + at) : identity<OP>();
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (g + u * G < left) {
#pragma unroll
      for (int i = 0; i < N; ++i) acc[u & 3] = fold<OP>(acc[u & 3], x[u].get(i));
    }
  acc[1] = fold<OP>(acc[1], rest);
  return fold<OP>(fold<OP>(acc[0], acc[1]), fold<OP>(acc[2], acc[3]));
}
template <int OP, int W>
__device__ __forceinline__ float fold_lanes(float a) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) a = fold<OP>(a, __shfl_xor(a, o, 64));
  return a;
}

// ROW: G lanes per row, 256 / G rows per block.
// G = 256: a row may be cut in `slices` slices of `slice` elements, one block each; `rows` then counts slices.
template <int OP, typename Tin, typename Tout, int G, bool VEC>
__global__ __launch_bounds__(256) void reduce_row_kernel(const Tin *in, Tout *out, int64_t rows, int64_t len, int64_t pitch, int slices = 1, int64_t slice = 0) {
  constexpr int RPB = 256 / G;
  const int g = threadIdx.x % G;
  const int64_t row = (int64_t)blockIdx.x * RPB + threadIdx.x / G;
  float a = identity<OP>();
  if (row < rows) {
    const Tin *p = in + row * pitch;
    if (G == 256 && slices > 1) {
      const int64_t r = row / slices, first = (row - r * slices) * slice;
      p = in + r * pitch + first;
      len = len - first < slice ? len - first : slice;
    }
    a = fold_row<OP, Tin, G, VEC, 1>(p, len, g);
  }
  a = fold_lanes<OP, (G < 64 ? G : 64)>(a);
  if constexpr (G == 256) {
    __shared__ float part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0 && row < rows)
      Elem<Tout>::store(out + row, fold<OP>(fold<OP>(part[0], part[1]), fold<OP>(part[2], part[3])));
  } else {
    if (g == 0 && row < rows) Elem<Tout>::store(out + row, a);
  }
}

template <int OP, typename Tin, typename Tout>
__global__ __launch_bounds__(256) void reduce_row_by_wave_kernel(const Tin *in, Tout *out, int64_t rows, int64_t len, int64_t pitch) {
  const int g = threadIdx.x % 64;
  const int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
  if (row >= rows) return;
  const float a = fold_lanes<OP, 64>(fold_row_by_wave<OP, Tin>(in + row * pitch, len, g));
  if (g == 0) Elem<Tout>::store(out + row, a);
}

// ROW without a workspace for the slices' results: one block folds all slices of its row in the same order, so that the
// result has the same bits.  Bound by the latency of what one block has in flight: four groups of 256 threads take
// the slices in turn, and their waves' results wait in LDS for kHeld slices at a time.
template <int OP, typename Tin, typename Tout>
__global__ __launch_bounds__(1024) void reduce_row_alone_kernel(const Tin *in, Tout *out, int64_t len, int64_t pitch, int slices, int64_t slice) {
  constexpr int kHeld = 1024;
  __shared__ __align__(16) float result[kMaxSlices];
  __shared__ float part[kHeld][4];
  const Tin *p = in + (int64_t)blockIdx.x * pitch;
  const int t = threadIdx.x & 255, wave = t >> 6;
  const bool first_lane = (threadIdx.x & 63) == 0;
  for (int s0 = 0; s0 < slices; s0 += kHeld) {
    const int n = min(slices - s0, kHeld);
    for (int s = threadIdx.x >> 8; s < n; s += 4) {
      const int64_t first = (s0 + s) * slice;
      const float a = fold_lanes<OP, 64>(fold_row<OP, Tin, 256, true, 2>(p + first, len - first < slice ? len - first : slice, t));
      if (first_lane) part[s][wave] = a;
    }
    __syncthreads();
    if ((int)threadIdx.x < n) {
      const float *w = part[threadIdx.x];
      result[s0 + threadIdx.x] = fold<OP>(fold<OP>(w[0], w[1]), fold<OP>(w[2], w[3]));
    }
    __syncthreads();
  }
  if (threadIdx.x < 256) {
    const float a = fold_lanes<OP, 64>(fold_row<OP, float, 256, true, 1>(result, slices, t));
    if (first_lane) part[0][wave] = a;
  }
  __syncthreads();
  if (threadIdx.x == 0) Elem<Tout>::store(out + blockIdx.x, fold<OP>(fold<OP>(part[0][0], part[0][1]), fold<OP>(part[0][2], part[0][3])));
}

// COL: out[o, i] (or partial[s, o, i]) = fold over r in this block's slice of in[o*sO + r*sR + i].
template <int OP, typename Tin, typename Tout, bool VEC, int kColTX>
__global__ __launch_bounds__(256) void reduce_col_kernel(const Tin *in, Tout *out, int64_t R, int64_t I, int64_t sO, int64_t sR,
                                                         int64_t rows_per_split, int64_t out_split_stride) {
  constexpr int N = VEC ? Vec16<Tin>::N : 1;
  constexpr int kColTY = 256 / kColTX;
  const int tx = threadIdx.x % kColTX, ty = threadIdx.x / kColTX;
  // (the last vector of a row that is not a whole number of them ends with the row: its first columns are folded
  // twice, by two threads that write the same values)
  const int64_t first = ((int64_t)blockIdx.x * kColTX + tx) * N, col = VEC && first < I && first + N > I ? I - N : first;
  const int64_t o = blockIdx.z;
  const int64_t r_begin = (int64_t)blockIdx.y * rows_per_split;
  int64_t r_end = r_begin + rows_per_split;
  if (r_end > R) r_end = R;
  float acc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = identity<OP>();
  if (col < I) {
    const Tin *p = in + o * sO + col;
    int64_t r = r_begin + ty;
    if constexpr (kColTX == kColTXShort) {
      // (Addresses by addition and lanes past the end by four selected words, not sixteen 64-bit products and branches:
      // the kernel is one cold pass over its own code, 1024 x 1000 bf16 between other kernels 5.1 -> 4.1 us, whatever
      // pages the code lies on.)
      constexpr int U = 16;
      const Tin *q = p + r * sR;
      const int64_t step = kColTY * sR;
      for (; r < r_end; r += U * kColTY, q += U * step) {
        const int n = (int)min((r_end - r + kColTY - 1) / kColTY, (int64_t)U);   // this lane's rows of the batch
        std::conditional_t<VEC, Vec16<Tin>, float> x[U];
        const Tin *at = q;
#pragma unroll
        for (int u = 0; u < U; ++u) {          // a lane past the end re-reads its last row and drops it
          if constexpr (VEC) x[u] = load16_any(at); else x[u] = Elem<Tin>::load(at);
          at += u + 1 < n ? step : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if constexpr (VEC) {
            uint32_t w[4];
            __builtin_memcpy(w, &x[u].raw, 16);
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = u < n ? w[i] : identity_word<OP, Tin>();
            __builtin_memcpy(&x[u].raw, w, 16);
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] = fold<OP>(acc[i], x[u].get(i));
          } else {
            acc[0] = fold<OP>(acc[0], u < n ? x[u] : identity<OP>());
          }
        }
      }
    } else if constexpr (VEC) {
      // Eight rows in flight per lane, then one batch of four and single ones (14795 x 296 fp32 22.7 -> 16.5 us, 16384 x 1024
      // bf16 14.5 -> 12.2 against four); four where the many narrow blocks of wide fp32 arrays keep memory busy as it is
      // (4000 x 8000 23.3, would be 24.3).  The single ones stay in the caches: where rows start off cache lines, a neighbour
      // wants the other part of the line (3000 x 2351 bf16 7.8 us, past the caches 9.5).
      constexpr int kBatch = sizeof(Tin) == 4 && kColTX == kColTXWide ? 4 : 8;
      auto batch = [&](auto count) __attribute__((always_inline)) {
        constexpr int U = decltype(count)::value;
        Vec16<Tin> x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = load16_any_nt(p + (r + u * kColTY) * sR);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < N; ++i) acc[i] = fold<OP>(acc[i], x[u].get(i));
        r += U * kColTY;
      };
      while (r + (kBatch - 1) * kColTY < r_end) batch(std::integral_constant<int, kBatch>{});
      if (kBatch > 4 && r + 3 * kColTY < r_end) batch(std::integral_constant<int, 4>{});
      for (; r < r_end; r += kColTY) {
        const Vec16<Tin> x = load16_any(p + r * sR);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = fold<OP>(acc[i], x.get(i));
      }
    } else {
      for (; r + 3 * kColTY < r_end; r += 4 * kColTY) {
        float x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = Elem<Tin>::load(p + (r + u * kColTY) * sR);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[0] = fold<OP>(acc[0], x[u]);
      }
      for (; r < r_end; r += kColTY) acc[0] = fold<OP>(acc[0], Elem<Tin>::load(p + r * sR));
    }
  }
  // The short shape folds its 16 row lanes per wave with butterflies first (lanes of one column
  // group are 4 apart), so that only one partial per wave goes through LDS.
  constexpr int kParts = kColTX == kColTXShort ? 4 : kColTY;
  __shared__ float part[kParts][kColTX * N + 1];
  if constexpr (kColTX == kColTXShort) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int off = kColTX; off < 64; off <<= 1) acc[i] = fold<OP>(acc[i], __shfl_xor(acc[i], off));
    if (threadIdx.x % 64 < kColTX) {
#pragma unroll
      for (int i = 0; i < N; ++i) part[threadIdx.x / 64][tx * N + i] = acc[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) part[ty][tx * N + i] = acc[i];
  }
  __syncthreads();
  // All threads fold: a column each (with eight bf16 columns per thread of one row lane, 32 threads had 64 values to read
  // one after the other: 64 x 179 bf16 2.7 us, 2.2 like this).
  Tout *q = out + (int64_t)blockIdx.y * out_split_stride + o * I;
#pragma unroll
  for (int c = threadIdx.x; c < kColTX * N; c += 256) {
    const int64_t f = ((int64_t)blockIdx.x * kColTX + c / N) * N, at = VEC && f < I && f + N > I ? I - N : f;
    if (at < I) {
      float v[kParts];                                       // folded as a tree: fewest roundings at full magnitude
#pragma unroll
      for (int y = 0; y < kParts; ++y) v[y] = part[y][c];
#pragma unroll
      for (int h = kParts / 2; h > 0; h /= 2)
#pragma unroll
        for (int y = 0; y < h; ++y) v[y] = fold<OP>(v[y], v[y + h]);
      Elem<Tout>::store(q + at + c % N, v[0]);
    }
  }
}

struct GenArgs {
  int nk;
  int64_t kshape[CHN_MAX_NDIM], kstr[CHN_MAX_NDIM];
  int64_t len, sR, total_out;
};

template <int OP, typename Tin, typename Tout>
__global__ __launch_bounds__(256) void reduce_gen_kernel(const Tin *in, Tout *out, GenArgs a) {
  int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= a.total_out) return;
  int64_t off = 0, rem = e;
  for (int d = a.nk - 1; d >= 0; --d) { off += (rem % a.kshape[d]) * a.kstr[d]; rem /= a.kshape[d]; }
  float acc = identity<OP>();
  for (int64_t r = 0; r < a.len; ++r) acc = fold<OP>(acc, Elem<Tin>::load(in + off + r * a.sR));
  Elem<Tout>::store(out + e, acc);
}

template <int OP, typename Tin, typename Tout>
chn_status launch_col(const Tin *in, Tout *out, const RPlan &p, int64_t O, int64_t R, int64_t I, int64_t sO, int64_t sR,
                      int split, int64_t rps, int64_t split_stride, bool vec, int tx, hipStream_t st) {
  if (!vec && tx != kColTXShort) tx = kColTXNarrow;
  const int n = vec ? 16 / (int)sizeof(Tin) : 1;
  const int64_t cpb = (int64_t)tx * n;
  dim3 grid((unsigned)((I + cpb - 1) / cpb), (unsigned)split, (unsigned)O);
  if (O > 65535) return fail(CHN_ERR_SHAPE, "reduce: outer extent %lld too large for the column kernel", (long long)O);
  if (vec && tx == kColTXShort) hipLaunchKernelGGL((reduce_col_kernel<OP, Tin, Tout, true, kColTXShort>), grid, dim3(256), 0, st, in, out, R, I, sO, sR, rps, split_stride);
  else if (vec && tx == kColTXWide) hipLaunchKernelGGL((reduce_col_kernel<OP, Tin, Tout, true, kColTXWide>), grid, dim3(256), 0, st, in, out, R, I, sO, sR, rps, split_stride);
  else if (vec && tx == kColTXMid) hipLaunchKernelGGL((reduce_col_kernel<OP, Tin, Tout, true, kColTXMid>), grid, dim3(256), 0, st, in, out, R, I, sO, sR, rps, split_stride);
  else if (vec) hipLaunchKernelGGL((reduce_col_kernel<OP, Tin, Tout, true, kColTXNarrow>), grid, dim3(256), 0, st, in, out, R, I, sO, sR, rps, split_stride);
  else if (tx == kColTXShort) hipLaunchKernelGGL((reduce_col_kernel<OP, Tin, Tout, false, kColTXShort>), grid, dim3(256), 0, st, in, out, R, I, sO, sR, rps, split_stride);
  else hipLaunchKernelGGL((reduce_col_kernel<OP, Tin, Tout, false, kColTXNarrow>), grid, dim3(256), 0, st, in, out, R, I, sO, sR, rps, split_stride);
  (void)p;
  return check_launch("reduce col");
}

template <int OP, typename Tin, typename Tout>
chn_status launch(const RPlan &p, const chn_array *in, const chn_array *out, void *ws, hipStream_t st) {
  const Tin *src = static_cast<const Tin *>(in->data);
  Tout *dst = static_cast<Tout *>(out->data);
  if (p.kind == KIND_ROW) {
    const int64_t rows = p.nk == 1 ? p.kshape[0] : 1;
    const int64_t pitch = p.nk == 1 ? p.kstr[0] : 0;
    const int n = 16 / (int)sizeof(Tin);
    const bool vec = p.len >= 4 * n;                        // (16-byte accesses at any element address)
    const bool cut = p.slices > 1 && cut_pays(rows, p.len, (int)sizeof(Tin));
    if (cut && !ws) {
      hipLaunchKernelGGL((reduce_row_alone_kernel<OP, Tin, Tout>), dim3((unsigned)rows), dim3(1024), 0, st, src, dst, p.len, pitch, p.slices, p.slice);
      return check_launch("reduce row");
    }
    if (cut) {
      float *part = static_cast<float *>(ws);
      hipLaunchKernelGGL((reduce_row_kernel<OP, Tin, float, 256, true>), dim3((unsigned)(rows * p.slices)), dim3(256), 0, st, src, part, rows * p.slices, p.len, pitch, p.slices, p.slice);
      CHN_TRY(check_launch("reduce row slices"));
      hipLaunchKernelGGL((reduce_row_kernel<OP, float, Tout, 256, true>), dim3((unsigned)rows), dim3(256), 0, st, part, dst, rows, (int64_t)p.slices, (int64_t)p.slices, 1, (int64_t)0);
      return check_launch("reduce row");
    }
#define CHN_ROW(G)                                                                                          \
  do {                                                                                                      \
    const int64_t blocks = (rows + (256 / G) - 1) / (256 / G);                                              \
    if (blocks > 0x7fffffff) return fail(CHN_ERR_SHAPE, "reduce: too many rows");                           \
    if (vec) hipLaunchKernelGGL((reduce_row_kernel<OP, Tin, Tout, G, true>), dim3((unsigned)blocks), dim3(256), 0, st, src, dst, rows, p.len, pitch, 1, (int64_t)0); \
    else hipLaunchKernelGGL((reduce_row_kernel<OP, Tin, Tout, G, false>), dim3((unsigned)blocks), dim3(256), 0, st, src, dst, rows, p.len, pitch, 1, (int64_t)0);    \
  } while (0)
    if (rows >= kWaveRows && p.len >= kWaveRowLen && p.len * (int64_t)sizeof(Tin) <= kWaveRowBytes) {
      if ((rows + 3) / 4 > 0x7fffffff) return fail(CHN_ERR_SHAPE, "reduce: too many rows");
      hipLaunchKernelGGL((reduce_row_by_wave_kernel<OP, Tin, Tout>), dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, src, dst, rows, p.len, pitch);
    } else if (p.len >= 2048 || rows < 512) CHN_ROW(256);
    else if (p.len > 64) CHN_ROW(64);
    else CHN_ROW(8);
#undef CHN_ROW
    return check_launch("reduce row");
  }
  if (p.kind == KIND_COL) {
    if (p.split == 1)
      return launch_col<OP, Tin, Tout>(src, dst, p, p.O, p.len, p.I, p.sO, p.sR, 1, p.len, 0, p.vec, p.tx, st);
    float *part = static_cast<float *>(ws);
    const int64_t OI = p.O * p.I;
    CHN_TRY((launch_col<OP, Tin, float>(src, part, p, p.O, p.len, p.I, p.sO, p.sR, p.split, p.rows_per_split, OI, p.vec, p.tx, st)));
    // Second pass over the [split, O * I] partials: a small array, so the time is one chain of
    // dependent load batches per lane; the narrow-in-columns block shape keeps that chain short.
    // Off the 16-byte grid it takes vectors from 2048 columns on only (9340 x 451 bf16 in all 10.1 us with, 8.2 without).
    const bool wide2 = OI / 4 >= 512 && p.split >= 16;
    return launch_col<OP, float, Tout>(part, dst, p, 1, p.split, OI, 0, OI, 1, p.split, 0, OI % 4 == 0 || OI >= 2048, wide2 ? kColTXWide : kColTXNarrow, st);
  }
  GenArgs a{};
  a.nk = p.nk; a.len = p.len; a.sR = p.sR; a.total_out = p.total_out;
  for (int d = 0; d < p.nk; ++d) { a.kshape[d] = p.kshape[d]; a.kstr[d] = p.kstr[d]; }
  const int64_t blocks = (p.total_out + 255) / 256;
  if (blocks > 0x7fffffff) return fail(CHN_ERR_SHAPE, "reduce: output too large");
  hipLaunchKernelGGL((reduce_gen_kernel<OP, Tin, Tout>), dim3((unsigned)blocks), dim3(256), 0, st, src, dst, a);
  return check_launch("reduce general");
}

template <typename Tin, typename Tout>
chn_status launch_op(int op, const RPlan &p, const chn_array *in, const chn_array *out, void *ws, hipStream_t st) {
  if (op == CHN_REDUCE_SUM) return launch<CHN_REDUCE_SUM, Tin, Tout>(p, in, out, ws, st);
  return launch<CHN_REDUCE_MAX, Tin, Tout>(p, in, out, ws, st);
}

}  // namespace

chn_status reduce_one_axis(int op, const chn_array *in, int axis, int keepdims, const chn_array *out,
                           void *ws, size_t ws_bytes, bool static_scratch, bool alone, chn_stream stream) {
  if (op != CHN_REDUCE_SUM && op != CHN_REDUCE_MAX) return fail(CHN_ERR_OP, "reduce: unknown op %d", op);
  RPlan p;
  CHN_TRY(make_rplan(in, axis, &p, alone));
  CHN_TRY(validate(out, "out", true));
  if (!is_float(out->dtype)) return fail(CHN_ERR_DTYPE, "reduce: out must be F32 or BF16");
  const int ax = axis < 0 ? axis + in->ndim : axis;
  const int ond = keepdims ? in->ndim : in->ndim - 1;
  if (out->ndim != ond) return fail(CHN_ERR_SHAPE, "reduce: out has ndim %d, expected %d", out->ndim, ond);
  for (int d = 0, od = 0; d < in->ndim; ++d) {
    if (d == ax) {
      if (keepdims) { if (out->shape[od] != 1) return fail(CHN_ERR_SHAPE, "reduce: kept axis must have length 1"); ++od; }
      continue;
    }
    if (out->shape[od] != in->shape[d]) return fail(CHN_ERR_SHAPE, "reduce: out dimension %d has length %lld, expected %lld", od, (long long)out->shape[od], (long long)in->shape[d]);
    ++od;
  }
  if (!is_contiguous(out)) return fail(CHN_ERR_STRIDE, "reduce: out must be contiguous");
  if (p.total_out == 0) return CHN_OK;
  hipStream_t st = as_stream(stream);
  if (p.kind == KIND_EMPTY) {
    const float v = op == CHN_REDUCE_SUM ? 0.0f : -INFINITY;
    const unsigned blocks = (unsigned)((p.total_out + 255) / 256);
    if (out->dtype == CHN_F32) hipLaunchKernelGGL((fill_kernel<float>), dim3(blocks), dim3(256), 0, st, static_cast<float *>(out->data), p.total_out, v);
    else hipLaunchKernelGGL((fill_kernel<bf16_raw>), dim3(blocks), dim3(256), 0, st, static_cast<bf16_raw *>(out->data), p.total_out, v);
    return check_launch("reduce fill");
  }
  if (p.kind == KIND_COL && p.ws_bytes > 0) {
    if (static_scratch) {
      // the per-device array stands in for the caller's workspace; nothing is allocated
      if (p.ws_bytes > kScratchBytes)
        return fail(CHN_ERR_WORKSPACE, "reduce (static scratch): this reduction needs %zu bytes of partial sums, the built-in buffer holds %zu; use chn_reduce_axis with a workspace",
                    p.ws_bytes, kScratchBytes);
      CHN_TRY(scratch_of_current_device(&ws));
    } else {
      CHN_TRY(check_ws(ws, ws_bytes, p.ws_bytes, "reduce"));
    }
  }
  if (p.kind == KIND_ROW && p.slices > 1) {
    if (static_scratch) {
      if (p.slice_bytes <= kScratchBytes) CHN_TRY(scratch_of_current_device(&ws));
      else ws = nullptr;
    } else if (!ws || reinterpret_cast<uintptr_t>(ws) % 256 || ws_bytes < p.slice_bytes) {
      ws = nullptr;                                           // (no room for the slices' results: one block per row)
    }
  }
  if (in->dtype == CHN_F32 && out->dtype == CHN_F32) return launch_op<float, float>(op, p, in, out, ws, st);
  if (in->dtype == CHN_BF16 && out->dtype == CHN_F32) return launch_op<bf16_raw, float>(op, p, in, out, ws, st);
  if (in->dtype == CHN_BF16 && out->dtype == CHN_BF16) return launch_op<bf16_raw, bf16_raw>(op, p, in, out, ws, st);
  return launch_op<float, bf16_raw>(op, p, in, out, ws, st);
}

// ---- several axes at once ---------------------------------------------------------------------------------
// CHN_AXES(mask) / CHN_AXIS_ALL are carried out as a sequence of single-axis reductions, last axis first,
// over fp32 intermediates in the caller's workspace: neighbouring reduced dimensions that are jointly
// contiguous are merged into one axis first (a full sum of a contiguous array is one axis: one long row).  A long axis
// that is no row (strided elements, say) and is folded into few results is cut in two (length = r x c: c elements per row
// first, then the r row results): the general kernel gives every result to one thread.
struct Pass {
  chn_array in, out;     // out: contiguous fp32 intermediate, or the caller's out for the last pass
  int axis;
  size_t ws_need;        // partial sums of the column kernel for this pass
};
struct MultiPlan {
  Pass pass[2 * CHN_MAX_NDIM];
  int n = 0;
  size_t tmp_bytes[2] = {0, 0};   // two intermediates that take turns
  size_t partial_bytes = 0;       // partial sums a pass needs ..
  size_t slice_bytes = 0;         // .. and what cutting long rows would use (optional), at the same place
  size_t tmp() const { return ((tmp_bytes[0] + 255) & ~size_t(255)) + ((tmp_bytes[1] + 255) & ~size_t(255)); }
  size_t required() const { return tmp() + partial_bytes; }
  size_t total() const { return tmp() + (partial_bytes > slice_bytes ? partial_bytes : slice_bytes); }
};

void set_contiguous(chn_array *a, int dtype) {
  int64_t st = dtype_size(dtype);
  a->dtype = dtype;
  for (int d = a->ndim - 1; d >= 0; --d) { a->strides[d] = st; st *= a->shape[d] > 0 ? a->shape[d] : 1; }
}

chn_status make_multi(const chn_array *in, int axis_code, MultiPlan *mp) {
  CHN_TRY(validate(in, "in", false));
  if (!is_float(in->dtype)) return fail(CHN_ERR_DTYPE, "reduce: input must be F32 or BF16");
  const int nd = in->ndim;
  if (nd < 1) return fail(CHN_ERR_NDIM, "reduce: input needs at least one dimension");
  int mask;
  if (axis_code == CHN_AXIS_ALL) mask = (1 << nd) - 1;
  else {
    mask = axis_code - CHN_AXES(0);
    if (mask <= 0 || (mask >> nd) != 0) return fail(CHN_ERR_AXIS, "reduce: axis set 0x%x out of range for %d dimensions", mask, nd);
  }
  // working copy of the view; reduced flag per dimension
  chn_array cur = *in;
  bool red[CHN_MAX_NDIM];
  for (int d = 0; d < nd; ++d) red[d] = (mask >> d) & 1;
  // merge neighbouring reduced dimensions that are jointly contiguous (or of length 1)
  for (int d = cur.ndim - 2; d >= 0; --d) {
    if (!(red[d] && red[d + 1])) continue;
    const bool joint = cur.shape[d + 1] == 1 || cur.shape[d] == 1 || cur.strides[d] == cur.strides[d + 1] * cur.shape[d + 1];
    if (!joint) continue;
    if (cur.shape[d + 1] == 1) cur.strides[d + 1] = cur.strides[d];     // keep the stride that matters
    cur.shape[d + 1] *= cur.shape[d];
    for (int e = d; e + 1 < cur.ndim; ++e) { cur.shape[e] = cur.shape[e + 1]; cur.strides[e] = cur.strides[e + 1]; red[e] = red[e + 1]; }
    --cur.ndim;
  }
  int64_t kept = 1;
  for (int d = 0; d < cur.ndim; ++d) if (!red[d]) kept *= cur.shape[d];
  // one pass per remaining reduced dimension, last first
  int which = 0;
  for (int d = cur.ndim - 1; d >= 0; --d) {
    if (!red[d]) continue;
    if (cur.shape[d] >= (1 << 20) && kept < 512 && cur.ndim < CHN_MAX_NDIM) {
      RPlan whole;
      chn_array probe = cur;
      if (!probe.data) probe.data = reinterpret_cast<void *>(uintptr_t(256));
      CHN_TRY(make_rplan(&probe, d, &whole, false));
      int64_t c = 0;
      for (int64_t t = 8192; t >= 1024; t -= 4) if (cur.shape[d] % t == 0) { c = t; break; }
      if (whole.kind != KIND_ROW && c) {
        for (int e = cur.ndim; e > d + 1; --e) { cur.shape[e] = cur.shape[e - 1]; cur.strides[e] = cur.strides[e - 1]; red[e] = red[e - 1]; }
        ++cur.ndim;
        cur.shape[d + 1] = c; cur.strides[d + 1] = cur.strides[d]; red[d + 1] = true;
        cur.shape[d] /= c; cur.strides[d] = cur.strides[d + 1] * c;
        ++d;
      }
    }
    Pass &ps = mp->pass[mp->n++];
    ps.in = cur;
    ps.axis = d;
    chn_array nxt = cur;
    for (int e = d; e + 1 < nxt.ndim; ++e) { nxt.shape[e] = nxt.shape[e + 1]; red[e] = red[e + 1]; }
    --nxt.ndim;
    set_contiguous(&nxt, CHN_F32);
    nxt.data = nullptr;                      // filled in when the workspace is known
    ps.out = nxt;
    RPlan rp;
    chn_array probe = ps.in;
    if (!probe.data) probe.data = reinterpret_cast<void *>(uintptr_t(256));   // (planning only looks at alignment)
    CHN_TRY(make_rplan(&probe, d, &rp, false));
    ps.ws_need = rp.kind == KIND_COL ? rp.ws_bytes : 0;
    if (ps.ws_need > mp->partial_bytes) mp->partial_bytes = ps.ws_need;
    if (rp.kind == KIND_ROW && rp.slice_bytes > mp->slice_bytes) mp->slice_bytes = rp.slice_bytes;
    bool last = true;                        // (the last pass writes the caller's array)
    for (int e = 0; e < d; ++e) last = last && !red[e];
    const size_t ob = last ? 0 : (size_t)numel(&nxt) * sizeof(float);
    if (ob > mp->tmp_bytes[which]) mp->tmp_bytes[which] = ob;
    which ^= 1;
    cur = nxt;
  }
  return CHN_OK;
}

chn_status reduce_axis_impl(int op, const chn_array *in, int axis, int keepdims, const chn_array *out,
                            void *ws, size_t ws_bytes, bool static_scratch, chn_stream stream) {
  if (axis != CHN_AXIS_ALL && axis < CHN_AXES(0)) return reduce_one_axis(op, in, axis, keepdims, out, ws, ws_bytes, static_scratch, true, stream);
  if (op != CHN_REDUCE_SUM && op != CHN_REDUCE_MAX) return fail(CHN_ERR_OP, "reduce: unknown op %d", op);
  MultiPlan mp;
  CHN_TRY(make_multi(in, axis, &mp));
  CHN_TRY(validate(out, "out", true));
  if (!is_float(out->dtype)) return fail(CHN_ERR_DTYPE, "reduce: out must be F32 or BF16");
  if (!is_contiguous(out)) return fail(CHN_ERR_STRIDE, "reduce: out must be contiguous");
  // expected shape of out
  const int nd = in->ndim;
  const int mask = axis == CHN_AXIS_ALL ? (1 << nd) - 1 : axis - CHN_AXES(0);
  int od = 0;
  for (int d = 0; d < nd; ++d) {
    const bool r = (mask >> d) & 1;
    if (r && !keepdims) continue;
    if (od >= out->ndim || out->shape[od] != (r ? 1 : in->shape[d]))
      return fail(CHN_ERR_SHAPE, "reduce: out dimension %d does not match the reduced shape", od);
    ++od;
  }
  if (od != out->ndim) return fail(CHN_ERR_SHAPE, "reduce: out has ndim %d, expected %d", out->ndim, od);
  if (numel(out) == 0) return CHN_OK;
  if (static_scratch) {
    if (mp.required() > kScratchBytes)
      return fail(CHN_ERR_WORKSPACE, "reduce (static scratch): this reduction needs %zu bytes of intermediates, the built-in buffer holds %zu; use chn_reduce_axis with a workspace",
                  mp.required(), kScratchBytes);
    if (mp.total() > 0) CHN_TRY(scratch_of_current_device(&ws));
    ws_bytes = kScratchBytes;
  } else {
    CHN_TRY(check_ws(ws, ws_bytes, mp.required(), "reduce"));
  }
  char *base = static_cast<char *>(ws);
  char *tmp[2] = {base, base ? base + ((mp.tmp_bytes[0] + 255) & ~size_t(255)) : nullptr};
  char *partial = base ? tmp[1] + ((mp.tmp_bytes[1] + 255) & ~size_t(255)) : nullptr;
  const void *src = in->data;
  for (int i = 0; i < mp.n; ++i) {
    Pass &ps = mp.pass[i];
    ps.in.data = const_cast<void *>(src);
    const bool last = i == mp.n - 1;
    if (last) { ps.out.data = out->data; set_contiguous(&ps.out, out->dtype); }
    else ps.out.data = tmp[i & 1];
    CHN_TRY(reduce_one_axis(op, &ps.in, ps.axis, 0, &ps.out, partial, base ? ws_bytes - mp.tmp() : 0, false, false, stream));
    src = ps.out.data;
  }
  return CHN_OK;
}


}  // namespace chn

extern "C" {

size_t chn_reduce_axis_workspace_bytes(const chn_array *in, int axis) {
  if (axis == CHN_AXIS_ALL || axis >= CHN_AXES(0)) {
    chn::MultiPlan mp;
    if (!in || chn::make_multi(in, axis, &mp) != CHN_OK) return 0;
    return mp.total();
  }
  chn::RPlan p;
  if (chn::make_rplan(in, axis, &p, true) != CHN_OK) return 0;
  return p.kind == chn::KIND_COL ? p.ws_bytes : p.kind == chn::KIND_ROW ? p.slice_bytes : 0;
}

chn_status chn_reduce_axis(int op, const chn_array *in, int axis, int keepdims, const chn_array *out,
                           void *ws, size_t ws_bytes, chn_stream stream) {
  return chn::reduce_axis_impl(op, in, axis, keepdims, out, ws, ws_bytes, false, stream);
}

chn_status chn_reduce_axis_static(int op, const chn_array *in, int axis, int keepdims, const chn_array *out,
                                  chn_stream stream) {
  return chn::reduce_axis_impl(op, in, axis, keepdims, out, nullptr, 0, true, stream);
}

}  // extern "C"
