// Internal launch entry points, one per kernel family.  Each returns 0 or -1
// (HIP launch error) and only enqueues work on the given stream.
#pragma once
#include "s2attn_device.h"

namespace s2 {

int launch_fwd_f32(const KArgs& a, hipStream_t st);
int launch_bwd_f32(const KArgs& a, hipStream_t st);        // dQ, dK and dV (or partials), delta included

int launch_fwd_bf16(const KArgs& a, hipStream_t st);
int launch_bwd_dkdv_bf16(const KArgs& a, hipStream_t st);  // delta must be ready
int launch_bwd_dq_bf16(const KArgs& a, hipStream_t st);
// two-waves-per-SIMD dK/dV kernel for the shapes dkdv_split_applies() accepts
bool dkdv_split_applies(const KArgs& a);
int launch_bwd_dkdv_split_bf16(const KArgs& a, hipStream_t st);   // a.ds_spill set: also stores the dS blobs
// dQ from the dS blobs the dK/dV kernel stored (same shapes as dkdv_split_applies)
int launch_bwd_dq_spill_bf16(const KArgs& a, hipStream_t st);

// delta[b,h,t] = sum_d dout[b,t,h,d] * o[b,t,h,d], fp32, and lse2
int launch_delta_bf16(const KArgs& a, hipStream_t st);
// dk = sum of the partials of all parts (same for dv), cast to the output type
int launch_combine_partials(const KArgs& a, int dtype, hipStream_t st);

// Number of tile sequences walked together (see decode_slot) for a kernel whose XCD holds
// `slots` workgroups at a time, and the sequence count padded to a multiple of it.
inline int interleave_for(int T, int slots) { return T >= slots ? 1 : (slots + T - 1) / T; }
inline int pad_to(int n, int il) { return (n + il - 1) / il * il; }

// Grid of a launch with n_seq sequences of T tiles under decode_block.
struct Grid {
  int blocks, il, n_seq;
};
inline Grid grid_of(int T, int n_seq, int slots) {
  const int each = (n_seq + 7) / 8;   // sequences of one XCD
  const int want = interleave_for(T, slots);
  const int il = want < each ? want : each;
  return Grid{8 * T * pad_to(each, il), il, n_seq};
}

}  // namespace s2
