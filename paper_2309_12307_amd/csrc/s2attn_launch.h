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

// Grid of a launch with n_seq sequences of T tiles, neighbouring `share` of which (a divisor of
// n_seq) read the same K and V, on XCDs that hold `slots` workgroups at a time.  A bundle is the
// largest piece of the `share` that deals every XCD the same number of sequences; one sequence
// where no piece does.
struct Grid {
  int blocks;
  Deal deal;
};
inline Grid grid_of(int T, int n_seq, int share, int slots) {
  int bundle = 1;
  for (int m = share; m > 1; --m)
    if (share % m == 0 && n_seq / m % 8 == 0) { bundle = m; break; }
  const int each = (n_seq / bundle + 7) / 8 * bundle;   // sequences of one XCD
  const int want = interleave_for(T, slots);
  // An XCD's sequences go in walks of `want` or more, as even as they can be: a last walk of one or two starts its
  // heaviest tiles when nothing is left to run beside them.  us, walks of `want` and even ones: forward, H = 32,
  // Hkv = 16, D = 64, N = 6144, G = 1536 (three sequences, 2 + 1 and 3) 70 and 49; H = 32, N = 2304, G = 768 (twelve,
  // 11 + 1 and 12) 32 and 25; backward, H = 8, N = 7168, G = 1792 127 and 106; H = 40, Hkv = 20, N = 2520, G = 1260 188
  // and 147.  Not where a sequence has few tiles and the last walk fills half the slots or more, as it then has little left
  // to lose: forward, H = 8, G = 384, N = 14976 (39 of three tiles, 22 + 17 and 39) 28.6 and 30.8; G = 256, N = 20480 (80
  // of two, 32 + 32 + 16 and 40 + 40) 34.3 and 36.9; with eight tiles 1.02 to 1.14 for even walks.  58 shapes of two to
  // twelve tiles: 1.09 (forward) and 1.03 (backward) in the mean over walks of `want`, worst 0.97.
  const bool uneven = T <= 4 && each > want && 2 * (each % want) >= want;
  const int walks = each > want ? each / want : 1;
  const int il = uneven ? want : (each + walks - 1) / walks;
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
