// The recurrent layer's whole sequence in one launch per pass, cut so that nothing leaves an XCD between two steps.
//
// The batch rows of a sequence never meet: cut along the batch, sixteen rows to each of the eight XCDs, every XCD walks
// through time by itself.  Its (up to 32) compute units share the hidden units out; each keeps its part of the recurrent
// matrix in registers and LDS from the first step to the last, and what they exchange every step goes through the L2 they
// share: a word written there and read by another compute unit of the XCD takes 0.25 us; past the L2s, as the kernels of
// lstm_seq.hip exchange, 0.55, and those take four such trips a step.
//
// Workgroup b belongs to group b % 8, and the dispatcher deals consecutive workgroups out over the XCDs.  That is not taken
// on trust: before the first step the workgroups meet (below), say which XCD they run on, and a group that does not share one
// exchanges at device scope instead, more slowly and with the same results.
//
// Every wait is bounded, as in lstm_seq.hip: after `spin_limit` polls a wave raises the status word and its workgroup leaves; the
// others run out of polls, or see the word, and leave too.
#include "lstm_cell.h"
#include "lstm_xcd.h"
#include "split.h"

#include <type_traits>

namespace chn {
namespace xcd {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float float2_any __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kThreads = 256;
// Cache policies of a buffer access.  What a store leaves in the XCD's L2 is there for its other compute units; a load has to get
// past the vector cache of its own, which the device scope does (sc1) and the workgroup scope (sc0) does not.
constexpr int kLoadXcd = 16, kStoreXcd = 0, kLoadDevice = 17, kStoreDevice = 17;
constexpr int kNowhere = 0x7f000000;                   // a byte offset past every resource, whatever is added: loads give zero
constexpr unsigned kAbsent = 0xffffffffu;              // what a word of h holds until its value arrives
constexpr int kMayCross = 0x7f6;                       // sched_barrier: everything but matrix instructions
constexpr float kUnscale = 1.0f / (kSplitScale * kSplitScale);

__device__ __forceinline__ __amdgpu_buffer_rsrc_t resource(const void *p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
// Loads and stores of what a group exchanges, at the scope its members share.
template <bool LOCAL> __device__ __forceinline__ chn_u32x4 load16(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, LOCAL ? kLoadXcd : kLoadDevice);
}
template <bool LOCAL> __device__ __forceinline__ void store16(__amdgpu_buffer_rsrc_t r, int off, const chn_u32x4 &v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, LOCAL ? kStoreXcd : kStoreDevice);
}
template <bool LOCAL> __device__ __forceinline__ void store4(__amdgpu_buffer_rsrc_t r, int off, unsigned v) {
  __builtin_amdgcn_raw_buffer_store_b32(v, r, off, 0, LOCAL ? kStoreXcd : kStoreDevice);
}
template <bool LOCAL> __device__ __forceinline__ void store_word(unsigned *p, unsigned v) {
  if constexpr (LOCAL) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned load_word(const unsigned *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// two neighbouring bfloat16 values, or an fp32 one, the word never kAbsent (a NaN of another payload then)
__device__ __forceinline__ unsigned present(unsigned v) { return v == kAbsent ? 0xffff7fffu : v; }
__device__ __forceinline__ unsigned present_f32(float v) { return __float_as_uint(v) == kAbsent ? 0x7fffffffu : __float_as_uint(v); }

// Eight k of one row or column as the matrix instruction reads them: one bfloat16 vector, or the three parts of eight fp32.
template <typename T> struct Parts;
template <> struct Parts<bf16_raw> {
  bf16x8 h;
  __device__ __forceinline__ void set(const chn_u32x4 &v) { h = __builtin_bit_cast(bf16x8, v); }
};
template <> struct Parts<float> {
  bf16x8 h, m, l;
  __device__ __forceinline__ void set(const chn_u32x4 &a, const chn_u32x4 &b, float scale) {
    chn_u32x4 hh, mm, ll;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t x, y, z;
      split2(__uint_as_float(e < 2 ? a[2 * e] : b[2 * e - 4]) * scale, __uint_as_float(e < 2 ? a[2 * e + 1] : b[2 * e - 3]) * scale, x, y, z);
      hh[e] = x; mm[e] = y; ll[e] = z;
    }
    h = __builtin_bit_cast(bf16x8, hh); m = __builtin_bit_cast(bf16x8, mm); l = __builtin_bit_cast(bf16x8, ll);
  }
};
// Most of U's parts into the accumulation registers, where the matrix instruction reads them as well: left to itself the
// register allocator of a kernel this full moves them about in every step (500 copies).
constexpr int kPinned = 25;
__device__ __forceinline__ void pin(Parts<float> &p, int i) {
  if (i < kPinned) asm volatile("" : "+a"(p.h), "+a"(p.m));
}
__device__ __forceinline__ floatx4 mma(const bf16x8 &a, const bf16x8 &b, const floatx4 &c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// Four words a lane, seen as rows of sixteen lanes by words: transposed, so that row i holds word i of rows 0 to 3.
__device__ __forceinline__ void swap16(unsigned &a, unsigned &b) {       // odd rows of a change places with even rows of b
  const auto v = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = v[0]; b = v[1];
}
__device__ __forceinline__ void swap32(unsigned &a, unsigned &b) {       // the upper half of a with the lower half of b
  const auto v = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = v[0]; b = v[1];
}
__device__ __forceinline__ void transpose_rows(unsigned (&w)[4]) {
  swap16(w[0], w[1]); swap16(w[2], w[3]);
  swap32(w[0], w[2]); swap32(w[1], w[3]);
}

// s_barrier without waiting for vector memory: LDS writes before it are visible after it, stores and prefetches stay in flight
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_vector_memory() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)
  asm volatile("" ::: "memory");
}
// What is computed from x after this is not moved out of a loop: a kernel whose registers are full of U has none for constants.
__device__ __forceinline__ void keep_here(int &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ bool given_up(const unsigned *status) { return __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u; }
__device__ __forceinline__ void give_up(unsigned *status) { __hip_atomic_store(status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Before the first step, and before anything but marks is written, all workgroups meet: the first one waits until every other has
// said that it is there, and on which XCD, and opens the walk; or somebody's patience runs out first, and nobody walks.  One
// word decides, so that all see the same: kOpen with a bit for every group that shares an XCD, or kCalledOff, and the kernels
// launched behind take over (two such grids on one device can each hold compute units the other waits for; then both leave here
// after some milliseconds).  Run by one wave; returns the word.
__device__ __forceinline__ unsigned meet(unsigned *state, unsigned *ids, int peers, int n_groups, int group, int idx, int lane, int patience, unsigned share) {
  const unsigned mine = 1u + (unsigned)__builtin_amdgcn_s_getreg(20 | (3 << 11));      // hardware register 20, four bits: the XCD
  if (lane == 0) __hip_atomic_store(ids + group * kMaxPeers + idx, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const bool first = group == 0 && idx == 0;
  unsigned verdict = kCalledOff;
#pragma unroll 1
  for (int spins = 0; spins < patience; ++spins) {
    if (first) {
      // eight lanes a group, four members each; ids[group] of the first member is what the others are compared with
      const int g = lane >> 3;
      bool there = true, same = true;
      const unsigned lead = g < n_groups ? load_word(ids + g * kMaxPeers) : mine;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = (lane & 7) * 4 + e;
        const unsigned v = g < n_groups && m < peers ? load_word(ids + g * kMaxPeers + m) : lead;
        there = there && v != 0u;
        same = same && v == lead;
      }
      if (__all(there)) {
        const unsigned long long eights = __ballot(same);
        verdict = kOpen;
        for (int i = 0; i < kXcds; ++i)
          if ((eights >> (8 * i) & 0xff) == 0xff) verdict |= share & 1u << i;
        break;
      }
    } else {
      const unsigned v = load_word(state);
      if (v != 0u) return v;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  unsigned found = 0u;
  if (lane == 0) __hip_atomic_compare_exchange_strong(state, &found, verdict, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  found = (unsigned)__builtin_amdgcn_readfirstlane((int)found);
  return found ? found : verdict;
}

// ---- forward -------------------------------------------------------------------------------------------------------------
// z_t = zx_t + bias + h_{t-1} U for the group's sixteen rows: the workgroup owns 8 S hidden units = 32 S gate columns.  The
// product is taken transposed, gate columns along the rows of the 16 x 16 result (2 S tiles) and batch rows along its
// columns, so that a lane ends up with the four gates of one unit.  The four waves share the contraction (every fourth 32 k): a
// wave reads its k of h_{t-1} straight into the registers the instruction takes, and the sums meet in LDS.
// h is its own message: what a step will write is filled with a bit pattern that no pair of values takes (kAbsent) three steps
// ahead, and a reader loads what it needs until no word of it holds the pattern.  No counter, no acknowledged store, no second trip.
// bf16: the message is the step's block of Hs itself, which nobody reads again after its step.
//
// fp32: U and h are multiplied as three bfloat16 parts each (split.h).  The high and middle parts of U stay in registers, the low
// parts in LDS; h is split by the lane that makes it and exchanged as parts, in the order the instruction reads them, through four
// blocks of the workspace that take turns (a reader that splits for itself needs more registers than there are).  Step t fills the
// block that step t - 1 read, and only behind its first barrier: there the four waves together have seen h_t of every member, which a
// member sends when it has read the block for the last time.  (One wave's poll does not tell: it covers every fourth 32 k.)
// Odd waves hold -U, so that the one-sided error of the instruction cancels.  A sum that is not finite (infinities, NaN,
// 2^80 and more) is taken again on fp32 values.
template <typename T, int S>
__global__ __launch_bounds__(kThreads, 1) void lstm_xcd_fwd_kernel(FwdArgs a) {
  constexpr bool kSplit = sizeof(T) == 4;
  constexpr int NK = 2 * S, TILES = 2 * S, E = (int)sizeof(T), PARTS = kSplit ? 3 : 1;
  constexpr int NLO = !kSplit ? 0 : NK * TILES < 35 ? NK * TILES : 35;   // low parts that lie in LDS (beside the sums it holds 35 a wave)
  constexpr int kLoBytes = 4 * NLO * 1024, kSumBytes = S * 3 * 2 * 1024;
  constexpr int kUse = kLoBytes + kSumBytes + S * 128 + 16, kBytes = kUse > 84 * 1024 ? kUse : 84 * 1024;   // more than half: one workgroup a compute unit
  __shared__ __attribute__((aligned(1024))) char lds[kBytes];
  bf16x8 *const lo = reinterpret_cast<bf16x8 *>(lds);
  floatx4 *const sums = reinterpret_cast<floatx4 *>(lds + kLoBytes);
  float *const bias = reinterpret_cast<float *>(lds + kLoBytes + kSumBytes);   // [gate][unit]
  int *const word = reinterpret_cast<int *>(lds + kUse - 16);   // [0], [1]: a wait of an even, odd step ran out; [2]: how the group met
  const int group = blockIdx.x % kXcds, idx = blockIdx.x / kXcds;
  const int b0 = group * kRows;
  if (b0 >= a.B) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;
  const int B = a.B, H = a.H, u0 = idx * 8 * S, n_ks = (H + 31) / 32;

  // ---- the workgroup's columns of U, once: tile p, row 4 x + g is gate g of unit u0 + 8 (p / 2) + 2 x + p % 2
  Parts<T> u[NK][TILES];
  {
    const __amdgpu_buffer_rsrc_t ur = resource(a.Ut, ((4 * (int64_t)H - 1) * a.ut_pitch + H) * E);
    const float scale = wave & 1 ? -kSplitScale : kSplitScale;
#pragma unroll
    for (int i = 0; i < NK; ++i)
#pragma unroll
      for (int p = 0; p < TILES; ++p) {
        const int unit = u0 + 8 * (p >> 1) + 2 * (r >> 2) + (p & 1), k = 32 * (wave + 4 * i) + 8 * q;
        const int off = unit < H && k < H ? (int)((((int64_t)(r & 3) * H + unit) * a.ut_pitch + k) * E) : kNowhere;
        if constexpr (kSplit) {
          u[i][p].set(load16<true>(ur, off), load16<true>(ur, off == kNowhere ? off : off + 16), scale);
          if (S == 3) pin(u[i][p], i * TILES + p);
          if (i * TILES + p < NLO) lo[(wave * NLO + i * TILES + p) * 64 + lane] = u[i][p].l;
        } else {
          u[i][p].set(load16<true>(ur, off));
        }
      }
  }
  // ---- this lane's part of the cell (waves below S): batch row b, units j and j + 1
  const int b = b0 + r, j = u0 + 8 * wave + 2 * q;
  const bool live = wave < S && b < B && j < H;
  float c_state[2] = {0.0f, 0.0f};
  // zx of the coming step, zero in lanes that hold no unit
  const int z_off = live ? (int)(((int64_t)b * a.zx_pitch + j) * 4) : kNowhere;
  u32x2 zn[4];
  auto fetch = [&](int t) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t zr = resource(a.zx + (int64_t)t * B * a.zx_pitch, ((int64_t)(B - 1) * a.zx_pitch + 4 * (int64_t)H) * 4);
#pragma unroll
    for (int g = 0; g < 4; ++g) zn[g] = __builtin_amdgcn_raw_buffer_load_b64(zr, z_off, g * H * 4, 0);
  };
  // Where this lane's pair of values goes in the message of block t (the h that step t reads), part by part.  All of a lane's
  // addresses are an offset inside a step's rows, the rest scalar; a lane that holds no unit has offsets outside.
  const int n_groups = (B + kRows - 1) / kRows, message = kSplit ? n_ks * PARTS * 1024 : (int)(((int64_t)(B - 1) * a.h_pitch + H) * E);
  const int h_off = live ? (int)(((int64_t)b * a.h_pitch + j) * E) : kNowhere, c_off = live ? (int)(((int64_t)b * a.c_pitch + j) * 4) : kNowhere;
  const int g_off = live ? (int)(((int64_t)b * a.g_pitch + j) * 4) : kNowhere;
  const int pair_off = kSplit ? (live ? (j >> 5) * PARTS * 1024 + ((j >> 3 & 3) * 16 + r) * 16 + (j & 7) * 2 : kNowhere) : h_off;
  auto block = [&](int t) __attribute__((always_inline)) {
    if constexpr (kSplit) return resource(a.xbuf + ((int64_t)(t & 3) * n_groups + group) * message, message);
    else return resource(static_cast<const T *>(a.Hs) + (int64_t)t * B * a.h_pitch, message);
  };
  auto mark = [&](int t) __attribute__((always_inline)) {
    if (t <= a.n_steps) {
      const __amdgpu_buffer_rsrc_t m = block(t);
#pragma unroll
      for (int part = 0; part < PARTS; ++part) store4<false>(m, pair_off + part * 1024, kAbsent);
    }
  };
  fetch(0);
  if (live) {
    c_state[0] = a.Cs[(int64_t)b * a.c_pitch + j]; c_state[1] = a.Cs[(int64_t)b * a.c_pitch + j + 1];
  }
  if ((int)threadIdx.x < 32 * S) {
    const int unit = u0 + threadIdx.x % (8 * S);
    bias[threadIdx.x] = a.bias && unit < H ? a.bias[threadIdx.x / (8 * S) * H + unit] : 0.0f;
  }
  if constexpr (kSplit) {
    mark(0);
    // k past the width: zeros that stay
    if (idx == 0)
      for (int w = threadIdx.x; w < 4 * PARTS * 64; w += kThreads) {
        const int l = w & 63, k = 32 * (n_ks - 1) + 8 * (l >> 4), rest = w >> 6;
        if (k >= H)
          for (int e = 0; e < 4; ++e)
            store_word<false>(reinterpret_cast<unsigned *>(a.xbuf + ((int64_t)(rest & 3) * n_groups + group) * message + ((n_ks - 1) * PARTS + (rest >> 2)) * 1024 + l * 16) + e, 0u);
      }
  }
  mark(1);
  mark(2);
  wait_vector_memory();                                // U, the first inputs; the marks are in place
  __syncthreads();
  if (wave == 0) {
    const unsigned m = meet(a.state, a.ids, a.peers, n_groups, group, idx, lane, a.patience, a.share);
    if (lane == 0) { word[0] = word[1] = 0; word[2] = (int)m; }
  }
  __syncthreads();
  const unsigned met = (unsigned)__builtin_amdgcn_readfirstlane(word[2]);
  if (met == kCalledOff) return;

  // rows past the batch repeat its last one: they feed columns of the result that nobody looks at
  const int row = b < B ? b : B - 1;
  const int in_off = kSplit ? wave * PARTS * 1024 + (q * 16 + row - b0) * 16 : (int)(((int64_t)row * a.h_pitch + 32 * wave + 8 * q) * E);

  auto walk = [&](auto scope) __attribute__((always_inline)) {
    constexpr bool LOCAL = decltype(scope)::value;
    auto send = [&](int t, float v0, float v1) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t m = block(t);
      if constexpr (kSplit) {
        unsigned hi, mid, low;
        split2(v0 * kSplitScale, v1 * kSplitScale, hi, mid, low);
        store4<LOCAL>(m, pair_off, present(hi));
        store4<LOCAL>(m, pair_off + 1024, present(mid));
        store4<LOCAL>(m, pair_off + 2048, present(low));
      } else {
        store4<LOCAL>(m, pair_off, present(pack_bf16(v0, v1)));
      }
    };
    if constexpr (kSplit) {
      const u32x2 h0 = __builtin_amdgcn_raw_buffer_load_b64(resource(a.Hs, ((int64_t)(B - 1) * a.h_pitch + H) * 4), h_off, 0, 0);
      send(0, __uint_as_float(h0[0]), __uint_as_float(h0[1]));
    }
#pragma unroll 1
    for (int t = 0; t < a.n_steps; ++t) {
      // ---- h_{t-1}, as it arrives (bf16: the caller's h_0 first); k past the width read as zeros
      const __amdgpu_buffer_rsrc_t hr = block(t);
      const bool marked = kSplit || t > 0;
      chn_u32x4 v[NK][PARTS];
      int from = in_off;
      keep_here(from);
      bool ok = false;
#pragma unroll 1
      for (int spins = 0; !marked || spins < a.spin_limit; ++spins) {
#pragma unroll
        for (int i = 0; i < NK; ++i) {
          if constexpr (kSplit) {
#pragma unroll
            for (int part = 0; part < PARTS; ++part) v[i][part] = load16<LOCAL>(hr, from + (4 * i * PARTS + part) * 1024);
          } else {
            v[i][0] = load16<LOCAL>(hr, 32 * (wave + 4 * i) + 8 * q < H ? from + 128 * i * E : kNowhere);
          }
        }
        asm volatile("" ::: "memory");
        unsigned most = 0;
#pragma unroll
        for (int i = 0; i < NK; ++i)
#pragma unroll
          for (int part = 0; part < PARTS; ++part) most = max(most, max(max(v[i][part][0], v[i][part][1]), max(v[i][part][2], v[i][part][3])));
        if (!marked || !__any(most == kAbsent)) { ok = true; break; }
        if ((spins & 255) == 255 && given_up(a.status)) break;
      }
      if (!ok && lane == 0) { word[t & 1] = 1; give_up(a.status); }
      // ---- what the next steps need: their inputs on the way, the marks three steps ahead (acknowledged by this wait one
      // step on, before the step is published after which a reader may look for them; fp32: behind the barrier)
      wait_vector_memory();
      u32x2 z[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) z[g] = zn[g];
      fetch(t + 1 < a.n_steps ? t + 1 : t);
      if constexpr (!kSplit) mark(t + 3);
      // ---- the product, two tiles at a time: 8 w .. 8 w + 7 are the units of wave w, to which the others hand their sums
      floatx4 own[2] = {floatx4{0, 0, 0, 0}, floatx4{0, 0, 0, 0}};
#pragma unroll
      for (int w = 0; w < S; ++w) {
        floatx4 acc[2] = {floatx4{0, 0, 0, 0}, floatx4{0, 0, 0, 0}};
        if constexpr (kSplit) {
          floatx4 acc1[2] = {floatx4{0, 0, 0, 0}, floatx4{0, 0, 0, 0}};
#pragma unroll
          for (int i = 0; i < NK; ++i) {
            const bf16x8 xh = __builtin_bit_cast(bf16x8, v[i][0]), xm = __builtin_bit_cast(bf16x8, v[i][1]), xl = __builtin_bit_cast(bf16x8, v[i][2]);
            const Parts<T> &u0_ = u[i][2 * w], &u1_ = u[i][2 * w + 1];
            const int f = i * TILES + 2 * w;
            const bf16x8 l0 = f < NLO ? lo[(wave * NLO + f) * 64 + lane] : u0_.l, l1 = f + 1 < NLO ? lo[(wave * NLO + f + 1) * 64 + lane] : u1_.l;
            acc1[0] = mma(u0_.h, xm, acc1[0]);
            acc1[1] = mma(u1_.h, xm, acc1[1]);
            acc1[0] = mma(u0_.m, xh, acc1[0]);
            acc1[1] = mma(u1_.m, xh, acc1[1]);
            acc[0] = mma(u0_.h, xh, acc[0]);
            acc[1] = mma(u1_.h, xh, acc[1]);
            acc1[0] = mma(u0_.m, xm, acc1[0]);
            acc1[1] = mma(u1_.m, xm, acc1[1]);
            acc1[0] = mma(u0_.h, xl, acc1[0]);
            acc1[1] = mma(u1_.h, xl, acc1[1]);
            acc1[0] = mma(l0, xh, acc1[0]);
            acc1[1] = mma(l1, xh, acc1[1]);
            __builtin_amdgcn_sched_barrier(kMayCross);
          }
          const float unscale = wave & 1 ? -kUnscale : kUnscale;
          acc[0] = (acc[0] + acc1[0]) * unscale;
          acc[1] = (acc[1] + acc1[1]) * unscale;
        } else {
#pragma unroll
          for (int i = 0; i < NK; ++i) {
            const bf16x8 xh = __builtin_bit_cast(bf16x8, v[i][0]);
            acc[0] = mma(u[i][2 * w].h, xh, acc[0]);
            acc[1] = mma(u[i][2 * w + 1].h, xh, acc[1]);
          }
          // the sums leave the accumulation registers here, not behind the branch below: there the compiler (ROCm 7.2) left out the
          // wait states between the last matrix instruction and the first read of its result
          asm volatile("" : "+v"(acc[0]), "+v"(acc[1]));
        }
        if (w == wave) {
          own[0] = acc[0]; own[1] = acc[1];
        } else {
          const int slot = w * 3 + (wave < w ? wave : wave - 1);
          sums[slot * 128 + lane] = acc[0];
          sums[slot * 128 + 64 + lane] = acc[1];
        }
      }
      lds_barrier();
      if (word[t & 1]) break;
      if constexpr (kSplit) mark(t + 3);
      if (wave < S) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          own[0] += sums[(wave * 3 + s) * 128 + lane];
          own[1] += sums[(wave * 3 + s) * 128 + 64 + lane];
        }
        if constexpr (kSplit) {
          float bad = 0.0f;                            // 0, or NaN
#pragma unroll
          for (int g = 0; g < 4; ++g) bad += 0.0f * own[0][g] + 0.0f * own[1][g];
          if (__builtin_expect(live && bad != 0.0f, 0)) {
            own[0] = own[1] = floatx4{0, 0, 0, 0};
            int jj = j;
            keep_here(jj);
            const float *ut = static_cast<const float *>(a.Ut) + (int64_t)jj * a.ut_pitch;
#pragma unroll 1
            for (int k = 0; k < H; ++k) {
              float h;
              if (t == 0) {                            // (the caller's h_0 may exceed what the parts hold)
                h = static_cast<const float *>(a.Hs)[(int64_t)b * a.h_pitch + k];
              } else {
                const int off = (k >> 5) * PARTS * 1024 + ((k >> 3 & 3) * 16 + r) * 16 + (k & 6) * 2, sh = k & 1 ? 0 : 16;
                h = 0.0f;
#pragma unroll
                for (int part = 2; part >= 0; --part)
                  h += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(hr, off + part * 1024, 0, LOCAL ? kLoadXcd : kLoadDevice) << sh & 0xffff0000u);
                h *= 1.0f / kSplitScale;
              }
              bool nan = true;
#pragma unroll
              for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                  own[e][g] = fmaf(h, ut[((int64_t)g * H + e) * a.ut_pitch + k], own[e][g]);
                  nan = nan && own[e][g] != own[e][g];
                }
              if (nan) break;                          // nothing that follows changes it
            }
          }
        }
        float hv[2];
        u32x2 gate[4], c_out;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          float s[4];
#pragma unroll
          for (int g = 0; g < 4; ++g) s[g] = (__uint_as_float(z[g][e]) + bias[g * 8 * S + 8 * wave + 2 * q + e]) + own[e][g];
          const float i = sigmoid_hw(s[0]), f = sigmoid_hw(s[1]), g = tanh_hw(s[2]), o = sigmoid_hw(s[3]);
          c_state[e] = f * c_state[e] + i * g;
          hv[e] = o * tanh_hw(c_state[e]);
          gate[0][e] = __float_as_uint(i); gate[1][e] = __float_as_uint(f); gate[2][e] = __float_as_uint(g); gate[3][e] = __float_as_uint(o);
          c_out[e] = __float_as_uint(c_state[e]);
        }
        send(t + 1, hv[0], hv[1]);
        if constexpr (kSplit)
          __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(hv[0]), __float_as_uint(hv[1])},
                                                resource(static_cast<const float *>(a.Hs) + (int64_t)(t + 1) * B * a.h_pitch, ((int64_t)(B - 1) * a.h_pitch + H) * 4), h_off, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b64(c_out, resource(a.Cs + (int64_t)(t + 1) * B * a.c_pitch, ((int64_t)(B - 1) * a.c_pitch + H) * 4), c_off, 0, 0);
        if (a.gates) {
          const __amdgpu_buffer_rsrc_t gr = resource(a.gates + (int64_t)t * B * a.g_pitch, ((int64_t)(B - 1) * a.g_pitch + 4 * (int64_t)H) * 4);
#pragma unroll
          for (int g = 0; g < 4; ++g) __builtin_amdgcn_raw_buffer_store_b64(gate[g], gr, g_off, g * H * 4, 0);
        }
      }
      lds_barrier();                                   // the sums have been read
    }
  };
  if (met >> group & 1) walk(std::true_type{});
  else walk(std::false_type{});
}

// ---- backward ------------------------------------------------------------------------------------------------------------
// dh_t = (gradient from above) + dz_{t+1} U^T, contracted over the 4 H gate columns, for the group's sixteen rows.  A workgroup's
// cell makes dz of its 8 S units; what it multiplies is another matter: the members stand in squares of four, a member gathers
// the dz of its square (the contraction: 128 S gate columns, a member's by each wave) and multiplies it with a quarter of U^T's
// units, by its place in the square.  So a step is two trips through the L2, dz to the four members of a square, then partial sums of dh
// to the owners of the units, one from every square, which they add in the squares' order.
// us a step at 128 rows, 672 units, bf16 / fp32: with every member multiplying its own dz with all of U^T and sending partial sums of all
// units to all members (one trip, but 1.2 MB a step and XCD each way, a wait for acknowledged stores and a flag) 4.4 and 6.6, now 3.1 and 6.3.
// A step is bound by its instructions, one wave a SIMD and about five cycles each (product and messages about half each), and the two trips.
// Values are their own arrival, as in the forward pass: four blocks of either kind of message take turns, what a block's next use will
// write holds kAbsent before.  Partial sums: the reader, the only one of those bytes, puts the marks back when it has read
// them.  dz: the sender marks its own words of the block of two steps ago once it has partial sums of this step: they were made, square
// by square, from dz of the step before, which a member sends when it has made its sums of two steps ago.  (A member without units
// sends no dz, but the sums it made of that block have been needed since.)  A wave waits for its marks before it sends its next dz; a block
// is used again two (dz) and four (sums) steps on, when everybody's dz of the step before has been waited for.
// tests/test_sequence_marks_backward.py is the protocol as a model.
template <typename T, int S>
__global__ __launch_bounds__(kThreads, 1) void lstm_xcd_bwd_kernel(BwdArgs a) {
  constexpr bool kSplit = sizeof(T) == 4;
  constexpr int TILES = 4 * S, E = (int)sizeof(T), PARTS = kSplit ? 3 : 1, PAIRS = kMaxPeers / 8;
  constexpr int NLO = !kSplit ? 0 : TILES * S < 27 ? TILES * S : 27;     // low parts that lie in LDS (beside the sums it holds 27 a wave)
  constexpr int kLoBytes = 4 * NLO * 1024, kSumBytes = TILES * 4 * 1024, SETS = kSplit ? 1 : 2;   // (two sets of sums: no barrier behind their use)
  constexpr int kUse = kLoBytes + SETS * kSumBytes + 16, kBytes = kUse > 84 * 1024 ? kUse : 84 * 1024;
  constexpr int kMessage = S * PARTS * 1024;                            // dz of a member
  __shared__ __attribute__((aligned(1024))) char lds[kBytes];
  bf16x8 *const lo = reinterpret_cast<bf16x8 *>(lds);
  floatx4 *const sums = reinterpret_cast<floatx4 *>(lds + kLoBytes);
  int *const word = reinterpret_cast<int *>(lds + kUse - 16);   // [0], [1]: a wait of an even, odd step ran out; [2]: how the group met
  const int group = blockIdx.x % kXcds, idx = blockIdx.x / kXcds;
  const int b0 = group * kRows;
  if (b0 >= a.B) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;
  const int B = a.B, H = a.H, u0 = idx * 8 * S, n_mt = H / 16, T_ = a.n_steps, G = a.peers, n_groups = (B + kRows - 1) / kRows;
  const int square = idx >> 2, quarter = (n_mt + 3) / 4, mt0 = (idx & 3) * quarter, n_tiles = min(n_mt - mt0, quarter);   // (n_tiles may be < 1)
  const int from = 4 * square + wave;                                    // the member whose dz this wave multiplies

  // ---- U, once: rows = units of the quarter (tile n), k-step s = unit 8 S from + 8 s + e of gate q
  Parts<T> u[TILES][S];
  {
    const __amdgpu_buffer_rsrc_t ur = resource(a.U, ((H - 1) * a.u_pitch + 4 * (int64_t)H) * E);
    const float scale = wave & 1 ? -kSplitScale : kSplitScale;
#pragma unroll
    for (int n = 0; n < TILES; ++n)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int row = 16 * (mt0 + n) + r, unit = from * 8 * S + 8 * s;
        const int off = n < n_tiles && unit < H ? (int)((row * a.u_pitch + q * H + unit) * E) : kNowhere;
        if constexpr (kSplit) {
          u[n][s].set(load16<true>(ur, off), load16<true>(ur, off == kNowhere ? off : off + 16), scale);
          if (S == 3) pin(u[n][s], n * S + s);
          if (n * S + s < NLO) lo[(wave * NLO + n * S + s) * 64 + lane] = u[n][s].l;
        } else {
          u[n][s].set(load16<true>(ur, off));
        }
      }
  }
  // ---- this lane's part of the cell (waves below S): batch row b, units j and j + 1
  const int b = b0 + r, j = u0 + 8 * wave + 2 * q;
  const bool live = wave < S && b < B && j < H;
  float dc[2] = {0.0f, 0.0f};
  typedef typename std::conditional<kSplit, u32x2, uint32_t>::type Pair;
  u32x2 gt[4], cprev;
  float cc[2] = {0.0f, 0.0f};
  Pair d_raw{};
  // Everything below is one wave a SIMD: an instruction costs five cycles whatever it does.  So what can be is an offset that stays
  // (all of a lane's, and `place` below; a kernel whose registers are full of U makes them anew) or a pointer that moves on.
  constexpr bool kFull = kSplit && S == 3;
  auto fresh = [&](int x) __attribute__((always_inline)) { if constexpr (kFull) keep_here(x); return x; };
  auto step_rows = [&](const void *p, int64_t pitch, int size, int t) __attribute__((always_inline)) { return static_cast<const char *>(p) + (int64_t)t * B * pitch * size; };
  const char *gates_t = step_rows(a.gates, a.g_pitch, 4, T_ - 1), *cs_t = step_rows(a.Cs, a.c_pitch, 4, T_ - 1), *dhs_t = step_rows(a.dHs, a.dh_pitch, E, T_ - 1);
  const char *dhs_out = dhs_t, *dz_out = step_rows(a.dZ, a.dz_pitch, E, T_ - 1);
  const int64_t gates_step = (int64_t)B * a.g_pitch * 4, cs_step = (int64_t)B * a.c_pitch * 4, dhs_step = (int64_t)B * a.dh_pitch * E, dz_step = (int64_t)B * a.dz_pitch * E;
  const int gates_bytes = (int)(((B - 1) * a.g_pitch + 4 * (int64_t)H) * 4), cs_bytes = (int)(((B - 1) * a.c_pitch + H) * 4);
  const int dhs_bytes = (int)(((B - 1) * a.dh_pitch + H) * E), dz_bytes_t = (int)(((B - 1) * a.dz_pitch + 4 * (int64_t)H) * E);
  auto lane_off = [&](int64_t pitch, int size) __attribute__((always_inline)) { return live ? (int)((b * pitch + fresh(j)) * size) : kNowhere; };
  auto fetch = [&]() __attribute__((always_inline)) {                    // the inputs of the step that the pointers are at: zeros in lanes that hold no unit
    const __amdgpu_buffer_rsrc_t gr = resource(gates_t, gates_bytes);
    const int at = lane_off(a.g_pitch, 4);
#pragma unroll
    for (int g = 0; g < 4; ++g) gt[g] = __builtin_amdgcn_raw_buffer_load_b64(gr, at, g * H * 4, 0);
    cprev = __builtin_amdgcn_raw_buffer_load_b64(resource(cs_t, cs_bytes), lane_off(a.c_pitch, 4), 0, 0);
    if constexpr (kSplit) d_raw = __builtin_amdgcn_raw_buffer_load_b64(resource(dhs_t, dhs_bytes), lane_off(a.dh_pitch, E), 0, 0);
    else d_raw = __builtin_amdgcn_raw_buffer_load_b32(resource(dhs_t, dhs_bytes), lane_off(a.dh_pitch, E), 0, 0);
    gates_t -= gates_step; cs_t -= cs_step; dhs_t -= dhs_step;
  };
  if (live) {
    if (a.dc_last) { dc[0] = a.dc_last[b * a.dcl_pitch + j]; dc[1] = a.dc_last[b * a.dcl_pitch + j + 1]; }
    cc[0] = a.Cs[((int64_t)T_ * B + b) * a.c_pitch + j]; cc[1] = a.Cs[((int64_t)T_ * B + b) * a.c_pitch + j + 1];
  }
  // ---- the messages of a step, [member][k-step][part][gate][16 rows][8 units] and [unit / 8][square][unit / 4 % 2][16 rows][4 units], an even number of squares (the one too many holds zeros), and this lane's
  // places in them, sixteen bytes each; lanes without a unit, and k-steps and units past the width, lie outside.  Rows past the batch repeat its last one.
  const int rows = B - b0 < kRows ? B - b0 : kRows, pairs = (G / 4 + 1) / 2;
  const int64_t dz_bytes = (int64_t)G * kMessage, sum_bytes = (int64_t)(H / 8) * pairs * 1024;
  auto dz_block = [&](int step) __attribute__((always_inline)) { return resource(a.xbuf + ((int64_t)(step & 3) * n_groups + group) * dz_bytes, dz_bytes); };
  auto sum_block = [&](int step) __attribute__((always_inline)) {
    return resource(a.xbuf + 4 * n_groups * dz_bytes + ((int64_t)(step & 3) * n_groups + group) * sum_bytes, sum_bytes);
  };
  const int j8 = u0 + 8 * wave;                                          // this wave's first unit
  auto dz_to = [&]() __attribute__((always_inline)) { return live ? idx * kMessage + wave * PARTS * 1024 + fresh(lane) * 16 : kNowhere; };
  // sums: lanes 16 q .. 16 q + 15 hold quad q / 2 of the squares of parity q % 2
  auto sums_at = [&](int pair) __attribute__((always_inline)) {
    const int l = fresh(lane);
    return ((j8 >> 3) * pairs + pair) * 1024 + (l >> 4 & 1) * 512 + (l >> 5) * 256 + min(l & 15, rows - 1) * 16;
  };
  const chn_u32x4 absent = {kAbsent, kAbsent, kAbsent, kAbsent};
  auto mark_dz = [&](int step, auto scope) __attribute__((always_inline)) {
    constexpr bool LOCAL = decltype(scope)::value;
    const __amdgpu_buffer_rsrc_t m = dz_block(step);
    const int to = dz_to();
#pragma unroll
    for (int part = 0; part < PARTS; ++part) store16<LOCAL>(m, to + part * 1024, absent);
  };
  auto mark_sums = [&](int step, auto scope) __attribute__((always_inline)) {
    constexpr bool LOCAL = decltype(scope)::value;
    const __amdgpu_buffer_rsrc_t m = sum_block(step);
    const int at = live ? sums_at(0) : kNowhere;
#pragma unroll
    for (int pair = 0; pair < PAIRS; ++pair) {
      const unsigned mark = 2 * pair + (fresh(lane) >> 4 & 1) < G / 4 ? kAbsent : 0u;
      store16<LOCAL>(m, pair < pairs ? at + pair * 1024 : kNowhere, chn_u32x4{mark, mark, mark, mark});
    }
  };
  if (wave < S) {
#pragma unroll 1
    for (int block = 0; block < 4; ++block) { mark_dz(block, std::false_type{}); mark_sums(block, std::false_type{}); }
  }
  fetch();
  wait_vector_memory();                                // U, the first inputs; the marks are in place
  __syncthreads();
  if (wave == 0) {
    const unsigned m = meet(a.state, a.ids, G, n_groups, group, idx, lane, a.patience, a.share);
    if (lane == 0) { word[0] = word[1] = 0; word[2] = (int)m; }
  }
  __syncthreads();
  const unsigned met = (unsigned)__builtin_amdgcn_readfirstlane(word[2]);
  if (met == kCalledOff || (u0 >= H && n_tiles < 1)) return;    // (a member that nobody waits for)

  auto walk = [&](auto scope) __attribute__((always_inline)) {
    constexpr bool LOCAL = decltype(scope)::value;
#pragma unroll 1
    for (int step = 0; step < T_; ++step) {
      const int t = T_ - 1 - step;
      float dzv[4][2] = {}, d[2] = {0.0f, 0.0f};
      bool ok = true;
      if (wave < S) {
        // what of the cell's backward does not depend on dh
        float k_o[2], k_c[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float tc = tanhf(cc[e]);
          k_o[e] = tc;
          k_c[e] = 1.0f - tc * tc;
        }
        if (step > 0) {
          // ---- the partial sums for this wave's units, one from every square
          const __amdgpu_buffer_rsrc_t xr = sum_block(step);
          chn_u32x4 part[PAIRS];
          const int at = j8 < H ? sums_at(0) : kNowhere;
          ok = false;
#pragma unroll 1
          for (int spins = 0; spins < a.spin_limit; ++spins) {
#pragma unroll
            for (int pair = 0; pair < PAIRS; ++pair) part[pair] = load16<LOCAL>(xr, pair < pairs ? at + pair * 1024 : kNowhere);
            asm volatile("" ::: "memory");
            unsigned most = 0;
#pragma unroll
            for (int pair = 0; pair < PAIRS; ++pair) most = max(most, max(max(part[pair][0], part[pair][1]), max(part[pair][2], part[pair][3])));
            if (!__any(most == kAbsent)) { ok = true; break; }
            if ((spins & 255) == 255 && given_up(a.status)) break;
          }
          if (!ok && lane == 0) { word[step & 1] = 1; give_up(a.status); }
          // the squares of each parity, then both: every lane keeps two of its four units
          floatx4 half = __builtin_bit_cast(floatx4, part[0]);
#pragma unroll
          for (int pair = 1; pair < PAIRS; ++pair) half += __builtin_bit_cast(floatx4, part[pair]);
          chn_u32x4 w = __builtin_bit_cast(chn_u32x4, half);
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            unsigned even = w[e], odd = w[2 + e];
            swap16(even, odd);
            d[e] = __uint_as_float(even) + __uint_as_float(odd);
          }
        }
        wait_vector_memory();                            // the marks of the step before are in place
        if constexpr (kSplit) { d[0] += __uint_as_float(d_raw[0]); d[1] += __uint_as_float(d_raw[1]); }
        else { d[0] += bf16_to_f32((bf16_raw)(d_raw & 0xFFFFu)); d[1] += bf16_to_f32((bf16_raw)(d_raw >> 16)); }
        // the total is what the cell sees and what is stored: in mixed precision that is the bf16 value
        if constexpr (!kSplit) {
          if (step > 0) { d[0] = bf16_to_f32(f32_to_bf16(d[0])); d[1] = bf16_to_f32(f32_to_bf16(d[1])); }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float i = __uint_as_float(gt[0][e]), f = __uint_as_float(gt[1][e]), g = __uint_as_float(gt[2][e]), o = __uint_as_float(gt[3][e]);
          const float c_before = __uint_as_float(cprev[e]);
          const float d_o = d[e] * k_o[e];
          const float dcv = dc[e] + d[e] * o * k_c[e];
          const float di = dcv * g, dg = dcv * i, df = dcv * c_before;
          cc[e] = c_before;
          dc[e] = dcv * f;
          dzv[0][e] = di * i * (1.0f - i);
          dzv[1][e] = df * f * (1.0f - f);
          dzv[2][e] = dg * (1.0f - g * g);
          dzv[3][e] = d_o * o * (1.0f - o);
        }
        // ---- dz to the members of the square, in the order the matrix instruction reads it: lanes 16 g .. 16 g + 15 hold eight units of gate g
        constexpr int WORDS = kSplit ? 2 : 1;
        unsigned dzw[WORDS][4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          if constexpr (kSplit) { dzw[0][g] = __float_as_uint(dzv[g][0]); dzw[WORDS - 1][g] = __float_as_uint(dzv[g][1]); }
          else dzw[0][g] = pack_bf16(dzv[g][0], dzv[g][1]);
        }
#pragma unroll
        for (int e = 0; e < WORDS; ++e) transpose_rows(dzw[e]);
        const bool sends = ok && step + 1 < T_;
        const __amdgpu_buffer_rsrc_t m = dz_block(step);
        const int to = sends ? dz_to() : kNowhere;
        if constexpr (kSplit) {
          chn_u32x4 part[3];
          float bad = 0.0f;                              // 0, or NaN
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            unsigned hi, mid, low;
            split2(__uint_as_float(dzw[0][k]) * kSplitScale, __uint_as_float(dzw[1][k]) * kSplitScale, hi, mid, low);
            bad = __builtin_fmaf(__uint_as_float(hi << 16), 0.0f, __builtin_fmaf(__uint_as_float(hi & 0xffff0000u), 0.0f, bad));
            part[0][k] = hi; part[1][k] = mid; part[2][k] = low;
          }
          if (__builtin_expect(bad != 0.0f, 0)) {
            // what the parts cannot hold: infinities, which make every sum that meets them be taken again, and the values' own halves in the
            // place of the other parts (kAbsent, two neighbours whose halves are all ones: one bit less)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const unsigned upper = dzw[0][k] >> 16 | (dzw[1][k] & 0xffff0000u), lower = (dzw[0][k] & 0xffffu) | dzw[1][k] << 16;
              part[0][k] = 0x7f807f80u;
              part[1][k] = upper == kAbsent ? 0xfffeffffu : upper;
              part[2][k] = lower == kAbsent ? 0xfffeffffu : lower;
            }
          }
#pragma unroll
          for (int p = 0; p < 3; ++p) store16<LOCAL>(m, to + p * 1024, part[p]);
        } else {
          store16<LOCAL>(m, to, chn_u32x4{present(dzw[0][0]), present(dzw[0][1]), present(dzw[0][2]), present(dzw[0][3])});
        }
        // what leaves the step, while dz is on its way; the marks are for steps two and four on
        if (step > 0) {
          const __amdgpu_buffer_rsrc_t dr = resource(dhs_out, dhs_bytes);
          const int at = lane_off(a.dh_pitch, E);
          if constexpr (kSplit) __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(d[0]), __float_as_uint(d[1])}, dr, at, 0, 0);
          else __builtin_amdgcn_raw_buffer_store_b32(pack_bf16(d[0], d[1]), dr, at, 0, 0);
        }
        const __amdgpu_buffer_rsrc_t zr = resource(dz_out, dz_bytes_t);
        const int out = live ? (int)((b * a.dz_pitch + (fresh(lane) >> 4) * H + j8) * E) : kNowhere;
        if constexpr (kSplit) {
#pragma unroll
          for (int e = 0; e < 2; ++e)
            __builtin_amdgcn_raw_buffer_store_b128(chn_u32x4{dzw[0][2 * e], dzw[1][2 * e], dzw[0][2 * e + 1], dzw[1][2 * e + 1]}, zr, out + 16 * e, 0, 0);
        } else {
          __builtin_amdgcn_raw_buffer_store_b128(chn_u32x4{dzw[0][0], dzw[0][1], dzw[0][2], dzw[0][3]}, zr, out, 0, 0);
        }
        if (step > 0 && step + 2 < T_) {
          mark_sums(step, scope);
          mark_dz(step + 2, scope);
        }
        dhs_out -= dhs_step; dz_out -= dz_step;
      }
      if (step + 1 == T_) break;
      // ---- the square's dz, as it arrives
      const __amdgpu_buffer_rsrc_t xr = dz_block(step);
      chn_u32x4 v[S][PARTS];
      const int l = fresh(lane);
      const int at = from * kMessage + (l >> 4) * 256 + min(l & 15, rows - 1) * 16;
      bool here = false;
#pragma unroll 1
      for (int spins = 0; spins < a.spin_limit; ++spins) {
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int part = 0; part < PARTS; ++part) v[s][part] = load16<LOCAL>(xr, from * 8 * S + 8 * s < H ? at + (s * PARTS + part) * 1024 : kNowhere);
        asm volatile("" ::: "memory");
        unsigned most = 0;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int part = 0; part < PARTS; ++part) most = max(most, max(max(v[s][part][0], v[s][part][1]), max(v[s][part][2], v[s][part][3])));
        if (!__any(most == kAbsent)) { here = true; break; }
        if ((spins & 255) == 255 && given_up(a.status)) break;
      }
      if (!here && lane == 0) { word[step & 1] = 1; give_up(a.status); }
      if (wave < S && t > 0) fetch();
      // ---- partial sums of the quarter's units, as many tiles at a time as there are registers for: tile 4 i + w is finished by
      // wave w
      constexpr int AT_ONCE = kFull ? 2 : kSplit ? 4 : TILES;
      floatx4 *const meet_at = sums + (SETS == 2 ? (step & 1) * (kSumBytes / 16) : 0);
#pragma unroll
      for (int n0 = 0; n0 < TILES; n0 += AT_ONCE) {
        if (kFull && n0 + AT_ONCE == TILES && n0 >= n_tiles) break;      // (up to 640 units nobody has the last two tiles: 128 x 544, 35 steps, 203 -> 190 us)
        floatx4 acc[AT_ONCE];
#pragma unroll
        for (int n = 0; n < AT_ONCE; ++n) acc[n] = floatx4{0, 0, 0, 0};
        if constexpr (kSplit) {
          floatx4 acc1[AT_ONCE], acc2[AT_ONCE];          // (products with a low part, in two chains)
#pragma unroll
          for (int n = 0; n < AT_ONCE; ++n) acc1[n] = acc2[n] = floatx4{0, 0, 0, 0};
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const bf16x8 xh = __builtin_bit_cast(bf16x8, v[s][0]), xm = __builtin_bit_cast(bf16x8, v[s][1]), xl = __builtin_bit_cast(bf16x8, v[s][2]);
#pragma unroll
            for (int n = 0; n < AT_ONCE; ++n) acc1[n] = mma(u[n0 + n][s].h, xm, acc1[n]);
#pragma unroll
            for (int n = 0; n < AT_ONCE; ++n) acc2[n] = mma(u[n0 + n][s].m, xh, acc2[n]);
#pragma unroll
            for (int n = 0; n < AT_ONCE; ++n) acc[n] = mma(u[n0 + n][s].h, xh, acc[n]);
#pragma unroll
            for (int n = 0; n < AT_ONCE; ++n) acc1[n] = mma(u[n0 + n][s].m, xm, acc1[n]);
#pragma unroll
            for (int n = 0; n < AT_ONCE; ++n) acc2[n] = mma(u[n0 + n][s].h, xl, acc2[n]);
#pragma unroll
            for (int n = 0; n < AT_ONCE; ++n) {
              const int f = (n0 + n) * S + s;
              acc1[n] = mma(f < NLO ? lo[(wave * NLO + f) * 64 + lane] : u[n0 + n][s].l, xh, acc1[n]);
            }
            __builtin_amdgcn_sched_barrier(kMayCross);
          }
          const float unscale = wave & 1 ? -kUnscale : kUnscale;
#pragma unroll
          for (int n = 0; n < AT_ONCE; ++n) acc[n] = (acc[n] + (acc1[n] + acc2[n])) * unscale;
        } else {
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const bf16x8 xh = __builtin_bit_cast(bf16x8, v[s][0]);
#pragma unroll
            for (int n = 0; n < AT_ONCE; ++n) acc[n] = mma(u[n][s].h, xh, acc[n]);
          }
        }
#pragma unroll
        for (int n = 0; n < AT_ONCE; ++n) meet_at[((n0 + n) * 4 + wave) * 64 + lane] = acc[n];
      }
      lds_barrier();
      if (word[step & 1]) break;
      {
        const __amdgpu_buffer_rsrc_t xw = sum_block(step + 1);
        auto send = [&](floatx4 acc, int n) __attribute__((always_inline)) {
          const int l = fresh(lane);
          const int to = n < n_tiles ? (2 * (mt0 + n) + (l >> 5)) * pairs * 1024 + square * 512 + (l & 31) * 16 : kNowhere;
          store16<LOCAL>(xw, to, chn_u32x4{present_f32(acc[0]), present_f32(acc[1]), present_f32(acc[2]), present_f32(acc[3])});
        };
        floatx4 sum[S];
        float bad = 0.0f;                                // 0, or NaN
#pragma unroll
        for (int i = 0; i < S; ++i) {
          const int n = 4 * i + wave;
          sum[i] = meet_at[n * 256 + lane];
#pragma unroll
          for (int s = 1; s < 4; ++s) sum[i] += meet_at[n * 256 + s * 64 + lane];
          if constexpr (kSplit) {
#pragma unroll
            for (int e = 0; e < 4; ++e) bad = n < n_tiles ? __builtin_fmaf(sum[i][e], 0.0f, bad) : bad;
          }
        }
        if (!kSplit || __builtin_expect(!__any(bad != 0.0f), 1)) {
#pragma unroll
          for (int i = 0; i < S; ++i) send(sum[i], 4 * i + wave);
        } else {
          // this wave's tiles again, on fp32 values; c = (member of the square, k-step, gate, unit)
#pragma unroll 1
          for (int n = wave; n < n_tiles; n += 4) {
            floatx4 acc = floatx4{0, 0, 0, 0};
            int at = min(r, rows - 1) * 16;
            keep_here(at);
#pragma unroll 1
            for (int c = 0; c < 4 * 32 * S; ++c) {
              const int m = 4 * square + c / (32 * S), k = c % (32 * S), unit = m * 8 * S + 8 * (k >> 5) + (k & 7), gate = (k >> 3) & 3, sh = k & 1 ? 0 : 16;
              if (unit >= H) continue;
              unsigned bits[3];
#pragma unroll
              for (int p = 0; p < 3; ++p)
                bits[p] = __builtin_amdgcn_raw_buffer_load_b32(xr, at, m * kMessage + ((k >> 5) * 3 + p) * 1024 + gate * 256 + (k & 6) * 2, LOCAL ? kLoadXcd : kLoadDevice) << sh & 0xffff0000u;
              const float hi = __uint_as_float(bits[0]);
              const float dz = hi * 0.0f != 0.0f ? __uint_as_float(bits[1] | bits[2] >> 16) : ((__uint_as_float(bits[2]) + __uint_as_float(bits[1])) + hi) * (1.0f / kSplitScale);
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[e] = fmaf(dz, static_cast<const float *>(a.U)[(int64_t)(16 * (mt0 + n) + 4 * q + e) * a.u_pitch + gate * H + unit], acc[e]);
            }
            send(acc, n);
          }
        }
      }
      if constexpr (SETS == 1) lds_barrier();            // the sums have been read
    }
  };
  if (met >> group & 1) walk(std::true_type{});
  else walk(std::false_type{});
  if (live && !word[0] && !word[1]) { a.dc0[b * a.dc0_pitch + j] = dc[0]; a.dc0[b * a.dc0_pitch + j + 1] = dc[1]; }
}

}  // namespace

#define CHN_XCD_LAUNCH(KERNEL)                                                                                     \
  do {                                                                                                             \
    const dim3 grid((unsigned)(kXcds * a.peers));                                                                  \
    const int s = units_of(a.H) / 8;                                                                               \
    if (bf16) {                                                                                                    \
      if (s == 1) hipLaunchKernelGGL((KERNEL<bf16_raw, 1>), grid, dim3(kThreads), 0, st, a);                       \
      else if (s == 2) hipLaunchKernelGGL((KERNEL<bf16_raw, 2>), grid, dim3(kThreads), 0, st, a);                  \
      else hipLaunchKernelGGL((KERNEL<bf16_raw, 3>), grid, dim3(kThreads), 0, st, a);                              \
    } else {                                                                                                       \
      if (s == 1) hipLaunchKernelGGL((KERNEL<float, 1>), grid, dim3(kThreads), 0, st, a);                          \
      else if (s == 2) hipLaunchKernelGGL((KERNEL<float, 2>), grid, dim3(kThreads), 0, st, a);                     \
      else hipLaunchKernelGGL((KERNEL<float, 3>), grid, dim3(kThreads), 0, st, a);                                 \
    }                                                                                                              \
  } while (0)

chn_status launch_fwd(const FwdArgs &a, bool bf16, hipStream_t st) {
  CHN_XCD_LAUNCH(lstm_xcd_fwd_kernel);
  return check_launch("lstm_seq_fwd");
}

chn_status launch_bwd(const BwdArgs &a, bool bf16, hipStream_t st) {
  CHN_XCD_LAUNCH(lstm_xcd_bwd_kernel);
  return check_launch("lstm_seq_bwd");
}

}  // namespace xcd
}  // namespace chn
