// The recurrent layer's whole-sequence kernels whose workgroups exchange inside one XCD's L2 (lstm_xcd.hip), as
// lstm_seq.hip's entry points see them.
#pragma once
#include "common.h"

namespace chn {
namespace xcd {

constexpr int kXcds = 8;                               // batch groups, one per XCD
constexpr int kRows = 16;                              // batch rows of a group
constexpr int kMaxPeers = 32;                          // workgroups of a group: one per compute unit of the XCD
constexpr int kMaxHidden = 24 * kMaxPeers;
constexpr int kPatience = 1 << 14;                     // polls (about 0.6 us each) after which a walk that has not begun is called off
// how the workgroups met: a bit for every group that shares an XCD beside the first, or nobody walks
constexpr unsigned kOpen = 1u << 30, kCalledOff = 1u << 31;

// The words of a workspace that are zero at launch: the status block of the kernels of lstm_seq.hip, with the state among it, their
// counters, then what they use for messages and these kernels for the members' ids, and messages of their own.
constexpr int kStateWord = 32, kFirstId = 128, kIdWords = kXcds * kMaxPeers, kWords = kFirstId + kIdWords;

struct FwdArgs {
  int B, H, n_steps, peers, spin_limit, patience;
  unsigned share;            // the groups (a bit each) that may exchange through an L2
  const float *zx; int64_t zx_pitch;
  const void *Ut; int64_t ut_pitch;
  const float *bias;
  void *Hs; int64_t h_pitch;
  float *Cs; int64_t c_pitch;
  float *gates; int64_t g_pitch;
  unsigned *status, *state, *ids;
  char *xbuf;
};
struct BwdArgs {
  int B, H, n_steps, peers, spin_limit, patience;
  unsigned share;
  const void *U; int64_t u_pitch;
  void *dHs; int64_t dh_pitch;
  const float *gates; int64_t g_pitch;
  const float *Cs; int64_t c_pitch;
  const float *dc_last; int64_t dcl_pitch;
  void *dZ; int64_t dz_pitch;
  float *dc0; int64_t dc0_pitch;
  unsigned *status, *state, *ids;
  char *xbuf;
};

// units of a workgroup: eight per 256 of the hidden width, so that at most 32 workgroups share a group's units
inline int units_of(int64_t H) { return H <= 256 ? 8 : H <= 512 ? 16 : 24; }
inline int peers_of(int64_t H) { return (int)((H + units_of(H) - 1) / units_of(H)); }
// the backward pass works in squares of four: members without units fill the last one
inline int peers_bwd(int64_t H) { return (peers_of(H) + 3) / 4 * 4; }
// whether the sizes fit
inline bool sizes_fit(int64_t B, int64_t H) { return B <= kXcds * kRows && H <= kMaxHidden; }
inline bool takes(int64_t B, int64_t H, int cus) { return sizes_fit(B, H) && cus >= kXcds * peers_bwd(H); }
// Steps from which a walk pays: U has to come into the registers, the workgroups have to meet, and the kernels that would take over
// are launched behind, which the first steps, cheaper each, have to earn back (us, the kernels of lstm_seq.hip against these: fp32
// forward 96 x 560 at one step 13.9 and 29.7, 32 x 528 at three 30.4 and 36.9, at four 39.4 and 40.7, 128 x 672 at four 53.0 and 44.8;
// fp32 backward 32 x 768 at five 56.2 and 58.8, at six 67.0 and 63.4, 8 x 384 at three 22.2 and 23.1, at four 28.5 and 26.4; bf16 backward
// 32 x 544 at four 24.9 and 26.0, at five 30.5 and 29.1, 64 x 224 at two 11.9 and 12.2, at three 15.9 and 14.0).  Measured at 8 to 128 rows,
// widths 64 to 768, one to twelve steps; few rows make those kernels' steps cheaper, more units a workgroup (8, 16, 24) make the start of
// these longer.  bf16 backward also decides against a call a step, which is the better start where little has to come in (8 x 64 at four
// steps 13.6 and 13.2, at three 12.1 and 9.3; 128 x 768 at three 29.9 and 28.6, at four 32.7 and 40.8).
inline int least_steps(bool backward, bool bf16, int64_t B, int64_t H) {
  static const int fwd[2][2][3] = {{{2, 3, 4}, {2, 3, 4}}, {{2, 3, 4}, {2, 2, 3}}};                            // [bf16][more than 64 rows]
  static const int bwd[2][3][3] = {{{3, 4, 6}, {3, 4, 5}, {3, 4, 4}}, {{4, 4, 5}, {3, 3, 4}, {3, 3, 4}}};      // [bf16][up to 32 rows, to 64, more]
  const int s = units_of(H) / 8 - 1;
  if (backward && bf16 && B <= 16 && H <= 64) return 5;
  return backward ? bwd[bf16][B <= 32 ? 0 : B <= 64 ? 1 : 2][s] : fwd[bf16][B > 64][s];
}
// bytes of the messages: fp32 exchanges the three parts of h through four blocks (of the widest row: the caller of the forward
// pass names no width), the backward pass dz (fp32: its three parts) and partial sums of dh through four blocks each
inline size_t fwd_messages(int64_t B) { return (size_t)((B + kRows - 1) / kRows * 4 * (kMaxHidden / 32) * 3 * 1024); }
inline size_t bwd_messages(int64_t B, int64_t H) {
  const int64_t g = peers_bwd(H);
  return 4 * (size_t)((B + kRows - 1) / kRows * (g * (units_of(H) / 8) * 3 * 1024 + (g / 4 + 1) / 2 * 2 * (H / 8) * 512));
}

chn_status launch_fwd(const FwdArgs &a, bool bf16, hipStream_t st);
chn_status launch_bwd(const BwdArgs &a, bool bf16, hipStream_t st);

}  // namespace xcd
}  // namespace chn
