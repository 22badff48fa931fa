// Internal launch entry points, one per kernel family.  Each returns 0 or -1
// (HIP launch error) and only enqueues work on the given stream.
#pragma once
#include "s2attn_device.h"

namespace s2 {

int launch_fwd_f32(const KArgs& a, hipStream_t st);
// dQ, dK and dV (or partials), delta included; dq_last: dQ in a launch of its own after dK/dV
int launch_bwd_f32(const KArgs& a, bool dq_last, hipStream_t st);
// the same for problems of few rows
int launch_fwd_f32_small(const KArgs& a, hipStream_t st);
int launch_bwd_f32_small(const KArgs& a, bool dq_last, hipStream_t st);

int launch_fwd_bf16(const KArgs& a, hipStream_t st);
int launch_bwd_dkdv_bf16(const KArgs& a, hipStream_t st);  // delta must be ready; a.ds_spill set: also stores the dS blobs
int launch_bwd_dq_bf16(const KArgs& a, hipStream_t st);
// most workgroups (D = 128, D = 64) that dK/dV and dQ share a launch with
constexpr int kOneLaunchBlocks = 6 * 256, kOneLaunchBlocks64 = 20 * 256;
// both in one launch for the shapes that gain by it; 1 and no launch for the others
int launch_bwd_both_bf16(const KArgs& a, hipStream_t st);
// few rows (D = 128): forward; dK/dV, dQ and delta in one launch (dq_last: dQ in a launch of its own after dK/dV)
bool fwd_is_small(const KArgs& a);
bool bwd_is_small(const KArgs& a);
int launch_fwd_small(const KArgs& a, hipStream_t st);
int launch_bwd_small(const KArgs& a, bool dq_last, hipStream_t st);
// head dimension 64, any shape (the three entry points above hand such calls on)
int launch_fwd_d64(const KArgs& a, hipStream_t st);
int launch_bwd_dkdv_d64(const KArgs& a, hipStream_t st);
int launch_bwd_both_d64(const KArgs& a, hipStream_t st);
int launch_bwd_dq_d64(const KArgs& a, hipStream_t st);
// dQ from the dS blobs the dK/dV kernel stored (same shapes)
int launch_bwd_dq_spill_bf16(const KArgs& a, hipStream_t st);

// delta[b,h,t] = sum_d dout[b,t,h,d] * o[b,t,h,d], fp32, and lse2
int launch_delta_bf16(const KArgs& a, hipStream_t st);
// dk = sum of the partials of all parts (same for dv), cast to the output type
int launch_combine_partials(const KArgs& a, int dtype, hipStream_t st);

// Number of tile sequences walked together (see decode_block) for a kernel whose XCD holds
// `slots` workgroups at a time, and the sequence count padded to a multiple of it.
inline int interleave_for(int T, int slots) { return T >= slots ? 1 : (slots + T - 1) / T; }
inline int pad_to(int n, int il) { return (n + il - 1) / il * il; }

// Sequences of the XCD that gets the most of n_seq: whole sequences are dealt round the eight.
inline int most_of_an_xcd(int n_seq) { return (n_seq + 7) / 8; }

// Sequences of T tiles that an XCD with `each` of them walks together, `want` or more (one walk where it has fewer).
// A last walk of one or two starts its heaviest tiles when nothing is left to run beside them, so the walks are even
// ones: forward, us, walks of `want` and these, H = 32, Hkv = 16, D = 64, N = 6144, G = 1536 (three sequences, 2 + 1 and 3)
// 70 and 49; H = 32, N = 2304, G = 768 (twelve, 11 + 1 and 12) 32 and 25; backward, H = 8, N = 7168, G = 1792 127 and
// 106; H = 40, Hkv = 20, N = 2520, G = 1260 188 and 147.  Where the even walks leave a last one less than three quarters
// full, or less full than walks of `want` do, the latter where theirs is three quarters full, longer ones otherwise
// (forward, walks of `want`, even ones, these: H = 8, Hkv = 1, N = 25536, G = 3648, Variant 2, seven sequences, three walks
// of 2 and a 1, two of 3 and a 1, 4 + 3, 206, 222 and 197; H = 40, Hkv = 10, D = 64, N = 10764, G = 5382, ten, 370, 380 and 336;
// H = 40, Hkv = 20, N = 17056, G = 1312, 65, ten of 6 and a 5, nine of 7 and a 2 321 and 328).
// Sequences of up to four tiles have little left to lose in a last walk that is half full (H = 8, G = 384, N = 14976: 39 of
// three, 22 + 17 and 39, 28.6 and 30.8; G = 256, N = 20480: 80 of two, 32 + 32 + 16 and 40 + 40, 34.3 and 36.9).  `crowded`, the
// four-wave forward, which reads K and V fastest for what it computes: nor have five or six in a second walk five eighths
// full where one walk of all would read twice the K and V that the XCD's L2 holds (G = 640, N = 16000, 25 of five, 13 + 12
// and 25, 36.7 and 38.9; G = 768, N = 13824, 18 of six, 11 + 7 and 18, 36.5 and 38.2; but where bundles share them, B = 2, H = 16,
// Hkv = 4, G = 714, 20 of six, 37.3 and 35.7; fp32, B = 2, H = 2, N = 14320, G = 358, Variant 2, backward, 238 and 214).
inline int walk_of(int T, int each, int bundle, int slots, bool crowded) {
  const int want = interleave_for(T, slots);
  if (each <= want) return each;
  const int rest = each % want, walks = each / want;
  if (rest == 0 || (T <= 4 && 2 * rest >= want)) return want;
  if (crowded && T <= 6 && walks == 1 && bundle == 1 && 8 * rest >= 5 * want) return want;
  auto last = [&](int il) { return (each - 1) % il + 1; };
  const int even = (each + walks - 1) / walks;
  if (4 * last(even) >= 3 * even && last(even) * want >= rest * even) return even;
  if (4 * rest >= 3 * want) return want;
  for (int il = even; il <= 2 * want; ++il)
    if (4 * last(il) >= 3 * il) return il;
  return last(even) * want >= rest * even ? even : want;
}

// Grid of a launch with n_seq sequences of T tiles, neighbouring `share` of which (a divisor of
// n_seq) read the same K and V, on XCDs that hold `slots` workgroups at a time.  A bundle is the
// largest piece of the `share` that deals every XCD the same number of sequences; one sequence
// where no piece does.
struct Grid {
  int blocks;
  Deal deal;
};
inline Grid grid_of(int T, int n_seq, int share, int slots, bool crowded = false) {
  int bundle = 1;
  for (int m = share; m > 1; --m)
    if (share % m == 0 && n_seq / m % 8 == 0) { bundle = m; break; }
  const int each = (n_seq / bundle + 7) / 8 * bundle;   // sequences of one XCD
  const int il = walk_of(T, each, bundle, slots, crowded);
  return Grid{8 * T * pad_to(each, il), Deal{n_seq, bundle, il, div_by(bundle), div_by(il), div_by(T * il)}};
}

// Launches `blocks` blocks of `threads` threads as kernel(args..., first_block).  A launch counts the work items of
// a dimension in 32 bits and runs what is left modulo 2^32, without an error.  Many tiny groups reach
// that (forward, G = 2: B * H * N = 2^25 rows), so a larger grid goes out in pieces, of a multiple of
// eight blocks as the XCD is the block number mod 8; a kernel adds first_block to its block id.
template <class Kernel, class... Args>
inline int launch_blocks(Kernel kernel, int blocks, int threads, hipStream_t st, const Args&... args) {
  const int piece = (int)(((1ll << 32) - 1) / threads / 8 * 8);
  for (int first = 0;; first += piece) {
    const int n = blocks - first < piece ? blocks - first : piece;
    hipLaunchKernelGGL(kernel, dim3(n), dim3(threads), 0, st, args..., first);
    if (hipGetLastError() != hipSuccess) return -1;
    if (n == blocks - first) return 0;
  }
}

}  // namespace s2
