// Shared between the host API and the kernels: the launch argument block and the
// shift/group index map of S2-Attn (LongLoRA Section 3.2, Algorithm 1).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace s2 {

// Element strides of one tensor: batch, token, head (the head-dim axis is contiguous).
struct TStride {
  long long b, t, h;
};

// Block and thread index (all launches are one-dimensional).  threadIdx and blockIdx go through
// functions of the device library that this build's floating-point flags keep from being inlined:
// a real call each, with its answer in a vector register even where it is the same for all lanes.
__device__ __forceinline__ int block_id() { return (int)__builtin_amdgcn_workgroup_id_x(); }
__device__ __forceinline__ int thread_id() { return (int)__builtin_amdgcn_workitem_id_x(); }

// Division of a number below 2^31 by a divisor known on the host: one multiplication on the
// scalar unit.  The compiler's division of two run-time numbers is some forty vector
// instructions, and a block's position takes about ten divisions before its first load.
struct Div {
  uint32_t mul, shift;
};
inline Div div_by(uint32_t d) {
  uint32_t shift = 0;
  while ((1ull << shift) < d) ++shift;
  return Div{(uint32_t)((((1ull << shift) - d) << 32) / d + 1), shift};
}
__device__ __forceinline__ int quot(int n, const Div& d) {
  return (int)(((uint32_t)(((uint64_t)(uint32_t)n * d.mul) >> 32) + (uint32_t)n) >> d.shift);
}

struct KArgs {
  const void* q; const void* k; const void* v;
  void* o; float* lse;                       // forward outputs / backward inputs
  const void* dout;
  void* dq; void* dk; void* dv;
  float* neg_delta;                          // (B,H,N) fp32: -delta, written by the pre-pass
  float* lse2;                               // (B,H,N) fp32: lse * log2(e), written by the pre-pass
  float* dkv_partial;                        // fp32 [dk, dv][parts][B,N,Hkv,D] or null
  void* ds_spill;                            // bf16 dS tiles handed from the dK/dV kernel to the dQ kernel, or null
  int c_begin, c_count;                      // kv heads [c_begin, c_begin + c_count) of this launch (spill path)
  TStride sq, sk, sv, sdq, sdk, sdv;         // q, k, v and their gradients may be strided views
  TStride so;                                // o and dout: contiguous (B,N,H,D)
  int B, N, H, Hkv, D, G;
  int r;                                     // H / Hkv
  int NG;                                    // N / G
  Div by_r, by_NG, by_parts, by_c_count;
  int shift;                                 // tokens, 0 <= shift < G
  int shifted_from;                          // heads >= shifted_from use the shifted partition
  int split;                                 // Variant 2: rows [0,split) | [split,G) of the wrap group; G = off
  int mixed;                                 // some kv head serves both head classes
  int parts;                                 // pieces the query heads of a kv head are cut into for dK/dV
  int ragged;                                // bf16 path: G % 128 != 0, shift % 64 != 0 or a Variant 2 split that
                                             // is not a multiple of 128 (partial tiles, wrap point inside a tile)
  float scale;                               // softmax scale
  float scale_log2;                          // scale * log2(e)
};

// Rolled position p of a head with shift s holds token (p + s) mod N
// (roll(x, -s) in Algorithm 1's first key line; both p and s are < N).
__device__ __forceinline__ int token_of(int p, int s, int N) {
  int t = p + s;
  return t >= N ? t - N : t;
}

// Element offset of row (batch b, token t, head h) of a tensor.
__device__ __forceinline__ size_t row_off(const TStride& s, int b, int t, int h) {
  return (size_t)((long long)b * s.b + (long long)t * s.t + (long long)h * s.h);
}

// A causal run: `len` consecutive rolled positions starting at `p0` inside which row i
// sees rows 0 .. i.  Normally a whole group (p0 = g * G, len = G); under Variant 2
// (Appendix B.3) the wrap-around group of a shifted head is two runs, [0, split) and
// [split, G) of the group.
struct Run {
  int p0, len;
};

// Token of row i of a run, with rows past its end (padding of a partial tile) clamped to
// the last row so that every load stays inside the tensor.
__device__ __forceinline__ int run_token(const KArgs& a, const Run& run, int i, int s) {
  return token_of(run.p0 + min(i, run.len - 1), s, a.N);
}

__device__ __forceinline__ int shift_of_head(const KArgs& a, int h) {
  return h >= a.shifted_from ? a.shift : 0;
}

// First visible key index for query row i of group g (0 except under Variant 2
// in the wrap-around group of a shifted head, Appendix B.3).
__device__ __forceinline__ int split_of_group(const KArgs& a, int g, int s) {
  return (s > 0 && g == a.NG - 1) ? a.split : a.G;   // a.split == G means "no split"
}

// How a launch deals its tile sequences out: bundles of `bundle` neighbouring sequences, which
// share K and V and so want one L2, go round the eight XCDs (as the block ids do).
struct Deal {
  int n_seq, bundle;
  int il;   // sequences of an XCD walked together
  Div by_bundle, by_il, by_span;   // span: T * il
};

// Reads one word of every 64 bytes of a kernel's KArgs and of the deal that follows them, and waits once.  The compiler
// loads arguments where they are first used, in three or four steps that each wait for memory as long as the CU has not
// seen them yet: 0.3 to 0.6 us of a launch (calls back to back, us without and with: forward, D = 64, N = 1024, H = 4,
// G = 256 7.4 and 7.0; few rows, N = 1024, H = 4 7.5 and 7.2, fp32, N = 256 4.7 and 4.1; dK/dV and dQ in one launch, N = 4096,
// H = 8, G = 1024 47.9 and 46.1; nothing at 100 us and more).  Kernels of two deals pass the second, and the 64 bytes that
// hold most of the first stay out: reading them too changes nothing (102 backward shapes: 1.000).  The few-row backwards
// spill 90 (bf16) and 48 (fp32) scalar registers with it, 75 and 40 without, and are 3 and 2 % faster all the same.  Not
// in the other backwards: those of fp32 and of D = 64 and the shared launch on partial tiles have no registers left for what
// is then kept (2 to 3 % slower), the separate dK/dV and dQ kernels are for large grids.
__device__ __forceinline__ void fetch_args(const KArgs& a, const Deal& deal) {
  asm volatile("" :: "s"(a.q), "s"(a.dv), "s"(a.sk.t), "s"(a.sdk.b), "s"(a.so.b), "s"(a.by_NG.mul), "s"(deal.by_span.shift));
}

// Block -> (sequence, rank): rank orders the T tiles of a sequence from heaviest (0) to lightest.
// `il` sequences of an XCD are walked together, heaviest tiles of all of them first: when a
// sequence has fewer tiles than the XCD has workgroup slots, several sequences are resident
// anyway, and this order hands every slot about the same total work (a plain
// sequence-by-sequence order leaves the slots that drew heavy tiles running at the end).
// False: the block has no tile (the grid is padded to whole bundles for every XCD and to a
// multiple of il).
__device__ __forceinline__ bool decode_block(int block, int T, const Deal& d, int& seq, int& rank) {
  const int slot = block >> 3;
  const int chunk = quot(slot, d.by_span);
  const int within = slot - chunk * T * d.il;
  rank = quot(within, d.by_il);
  const int y = chunk * d.il + within - rank * d.il;
  const int yb = quot(y, d.by_bundle);
  seq = (yb * 8 + (block & 7)) * d.bundle + y - yb * d.bundle;
  return seq < d.n_seq;
}

// Sequence number -> (batch, head, group), query heads of one (kv head, group) next to each other.
struct HeadPos {
  int b, c, h, g;
};
__device__ __forceinline__ HeadPos head_of_seq(const KArgs& a, int seq) {
  HeadPos p;
  const int t = quot(seq, a.by_r);
  const int u = quot(t, a.by_NG);
  p.g = t - u * a.NG;
  p.b = quot(u, a.by_c_count);
  p.c = a.c_begin + u - p.b * a.c_count;
  p.h = p.c * a.r + seq - t * a.r;
  return p;
}

// The same for dK/dV: (batch, kv head, group, part of the kv head's query heads).
struct KvPos {
  int b, c, g, part;
};
__device__ __forceinline__ KvPos kv_of_seq(const KArgs& a, int seq) {
  KvPos p;
  const int t = quot(seq, a.by_parts);
  p.part = seq - t * a.parts;
  const int u = quot(t, a.by_NG);
  p.g = t - u * a.NG;
  p.b = quot(u, a.by_c_count);
  p.c = a.c_begin + u - p.b * a.c_count;
  return p;
}

// Query heads [h_lo, h_lo + n) of part `part` of kv head c, all of one class, and their shift.
// A kv head with both classes gives the first parts / 2 parts to the unshifted heads (so parts
// is at least 2 there); a part may be empty.
__device__ __forceinline__ void part_heads(const KArgs& a, int c, int part, int& h_lo, int& n, int& shift) {
  int lo = c * a.r, hi = lo + a.r, p = part, np = a.parts;
  if (np == 1) {
    h_lo = lo;
    n = a.r;
    shift = lo >= a.shifted_from ? a.shift : 0;
    return;
  }
  const int f = min(max(a.shifted_from, lo), hi);
  const bool both = f > lo && f < hi;
  if (both) {
    const int n0 = np / 2;
    if (p < n0) { hi = f; np = n0; } else { lo = f; p -= n0; np -= n0; }
  }
  h_lo = __builtin_amdgcn_readfirstlane(lo + (hi - lo) * p / np);
  n = __builtin_amdgcn_readfirstlane(lo + (hi - lo) * (p + 1) / np - h_lo);
  shift = lo >= a.shifted_from ? a.shift : 0;
}

// ---- dS hand-over between the two backward kernels (tile-aligned shapes only).
// The dK/dV kernel stores dS = P * (dP - delta) of every (64 queries x 128 keys) tile it
// visits as one 16 KB blob, exactly as its waves hold it: [key block kb 0..3][operand f 0..3]
// [lane 0..63][8 bf16], where lane = 32 g + (key % 32) of the wave that owns keys
// 32 kb .. 32 kb + 31, and element e of the lane's f-th packed operand is query
// 32 (f / 2) + 16 (f % 2) + 8 (e / 4) + 4 g + (e % 4) of the tile.  Every store instruction
// of a wave therefore writes 1 KB of consecutive bytes.  Seen as a matrix with one row per
// key and the 64 queries along the columns in the order (f, g, e), the column index within
// every 16 queries is the query index with bits 2 and 3 exchanged.  The dQ kernel reads the
// blobs back instead of recomputing S and dP.
// Blobs of one (batch, query head, group) are ordered by key tile jt (128 keys), then by
// query tile it = 0, 1, ... counted from the diagonal (query rows 128 jt + 64 it ...); a key
// tile has 2 (T - jt) query tiles when the group has T key tiles.
constexpr int kDsBlobBytes = 64 * 128 * 2;
__host__ __device__ inline long long ds_blobs_per_group(int T) { return (long long)T * (T + 1); }
__host__ __device__ inline long long ds_blob_index(int T, int jt, int it) {
  return (long long)jt * (2 * T - jt + 1) + it;
}
// Query row (within its 16) of column `col` (within its 16) of a blob, and back: bits 2 and 3
// exchanged.
__host__ __device__ inline int ds_col_query(int col) {
  return (col & ~12) | ((col & 4) << 1) | ((col & 8) >> 1);
}

// Kernels built for partial tiles treat Variant 2 by running the two halves of the
// wrap-around group as causal runs of their own: tile index `t` of the group (tiles of
// `tile` rows, first run's tiles first) -> the run and the tile index inside it.  Returns
// false when the group has no such tile (the grid is sized for the worst case).
__device__ __forceinline__ bool run_of_tile(const KArgs& a, int g, int s, int tile, int& t, Run& run) {
  run.p0 = g * a.G;
  run.len = a.G;
  const int split = split_of_group(a, g, s);
  if (split < a.G) {
    const int t_first = (split + tile - 1) / tile;
    if (t < t_first) {
      run.len = split;
    } else {
      t -= t_first;
      run.p0 += split;
      run.len = a.G - split;
    }
  }
  return t * tile < run.len;
}

// Tiles of `tile` rows that a group needs at most under run_of_tile.
inline int ragged_tiles(const KArgs& a, int tile) {
  const int whole = (a.G + tile - 1) / tile;
  if (a.split >= a.G) return whole;
  const int two = (a.split + tile - 1) / tile + (a.G - a.split + tile - 1) / tile;
  return two > whole ? two : whole;
}

}  // namespace s2
