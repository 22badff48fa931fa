// bf16 S2-Attn for head dimension 64: forward, dK/dV and dQ kernels for gfx950.  Any even group
// size, any shift: a block works inside one causal run (run_of_tile), the shift is row addressing.
//
// The products, operand feedback and online softmax are those of the 128-wide kernels.  What
// differs is the balance: per (query, key) pair the exponentials and conversions are the same and
// the matrix work is half, so vector and matrix unit are about equally loaded (64 keys x 32
// queries, forward: 16 MFMAs = 512 cycles against 96 vector instructions and 32 exp2 = 640), and
// accumulators and register operands are half as large.  So no wave needs to be given a role of
// its own: several independent workgroups per CU fill the one unit while their neighbours use the
// other.  LDS tile rows are 128 bytes, two to a 256-byte bank row (tile_off64).
//
// N = 32768, H = 32, G = 8192 against the 128-wide kernels with the upper half of every row left
// out: forward 1516 -> 1236 us (matrix unit busy 54 % of the time at a clock of 1.6 GHz), dK/dV 3082 ->
// 2198 us (51 % at 1.9 GHz), dQ 1866 -> 1542 us (64 % at 1.6 GHz, the power limit).
#include "s2attn_bf16_common.h"
#include "s2attn_device.h"
#include "s2attn_launch.h"

namespace s2 {
namespace {

constexpr int DH = 64;
constexpr int kRow = DH * 2;            // bytes of a tile row
constexpr int kTR = 64;                 // rows per staged tile
constexpr int kTile = kTR * kRow;       // 8 KB
constexpr int kOwn = 128;               // rows a workgroup owns, 32 per wave

// Tile rows 2R and 2R + 1 share the 256-byte LDS row R; its eight chunk columns are XOR-permuted
// by a function of R mod 8 that takes every value (16 rows of one chunk column hit all banks) and
// differs in bit 2 between neighbouring R (4 rows x 64 bytes of a transposing read do too).
__device__ __forceinline__ int swz64(int R) { return ((R & 1) << 2) | ((R >> 1) & 3); }
__device__ __forceinline__ int tile_off64(int row, int chunk) {
  return (row >> 1) * 256 + ((row & 1) << 7) + ((chunk ^ swz64(row >> 1)) << 4);
}

struct Offsets64 {
  int rm[4];      // row-major fragment k: elements [16k + 8g, +8) of row l % 32
  int tr[2][2];   // transposed fragment, column block cb: rows 4g + L/4 and that + 8
};
__device__ __forceinline__ Offsets64 lane_offsets64(int lane) {
  Offsets64 o;
  const int l32 = lane & 31, g32 = lane >> 5, L = lane & 15;
#pragma unroll
  for (int k = 0; k < 4; ++k) o.rm[k] = tile_off64(l32, 2 * k + g32);
  const int row = 4 * g32 + (L >> 2);
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    const int col = 32 * cb + (lane & 16) + 4 * (L & 3);
    o.tr[cb][0] = tile_off64(row, col >> 3) + (col & 7) * 2;
    o.tr[cb][1] = tile_off64(row + 8, col >> 3) + (col & 7) * 2;
  }
  return o;
}
template <int ROW0>   // a multiple of 16
__device__ __forceinline__ bf16x8 rm64(const char* tile, const Offsets64& o, int k) {
  return *reinterpret_cast<const bf16x8*>(tile + o.rm[k] + ROW0 * kRow);
}
template <int ROW0>
__device__ __forceinline__ bf16x8 tr64(const char* tile, const Offsets64& o, int cb) {
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(S2_LDS(bf16x4, tile + o.tr[cb][0] + ROW0 * kRow));
  const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(S2_LDS(bf16x4, tile + o.tr[cb][1] + ROW0 * kRow));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Staging of 64-row tiles of two tensors by four waves: wave w, pass p fills the 8 tile rows from
// 8w + 32p (1 KB of LDS per tensor); a lane fetches the chunk that the layout places at its slot.
struct Stager {
  int row;            // this lane's row in pass 0
  uint32_t chunk;     // byte offset of its chunk in the row
  uint32_t lane_x, lane_y;   // row and chunk as byte offsets into the two tensors
};
__device__ __forceinline__ Stager stager(int w, int lane, uint64_t x_row_bytes, uint64_t y_row_bytes) {
  Stager st;
  const int R = 4 * w + (lane >> 4);
  st.row = 2 * R + ((lane >> 3) & 1);
  st.chunk = (uint32_t)(((lane & 7) ^ swz64(R)) << 4);
  st.lane_x = (uint32_t)(st.row * x_row_bytes) + st.chunk;
  st.lane_y = (uint32_t)(st.row * y_row_bytes) + st.chunk;
  return st;
}
// Rows t0 .. t0 + 63 of the run.  64 consecutive tokens (all tiles but a run's last one and one at
// the wrap of the roll) take a scalar base; otherwise every row finds its own token, rows past
// the end of the run repeating its last row.
__device__ __forceinline__ void stage_pair(const KArgs& a, const Run& run, int s, int t0, const Stager& st, int w,
                                           uint64_t x_head, uint64_t x_row_bytes, uint64_t y_head,
                                           uint64_t y_row_bytes, uint32_t lds_x, uint32_t lds_y) {
  const int p = run.p0 + t0 + s;
  if (t0 + kTR <= run.len && (p + kTR <= a.N || p >= a.N)) {
    const uint32_t tok0 = (uint32_t)(p >= a.N ? p - a.N : p);
    const uint64_t xb = x_head + tok0 * x_row_bytes, yb = y_head + tok0 * y_row_bytes;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      dma16s(xb + q * 32 * x_row_bytes, st.lane_x, lds_x + (w + 4 * q) * 1024);
      dma16s(yb + q * 32 * y_row_bytes, st.lane_y, lds_y + (w + 4 * q) * 1024);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint64_t tok = (uint64_t)run_token(a, run, t0 + st.row + 32 * q, s);
      dma16(reinterpret_cast<const char*>(x_head + tok * x_row_bytes + st.chunk), lds_x + (w + 4 * q) * 1024);
      dma16(reinterpret_cast<const char*>(y_head + tok * y_row_bytes + st.chunk), lds_y + (w + 4 * q) * 1024);
    }
  }
}

// A wave's 32 x 64 result (rows lane-indexed, columns register-indexed) through its own 4 KB of
// LDS, then to rows [row0, row0 + 32) of the run: `wave_rows` fills the LDS, `store_rows` (after
// a barrier) writes 16 bytes per lane.
__device__ __forceinline__ void wave_rows(char* region, const f32x16 (&acc)[2], float mul, int l32, int g32) {
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int vv = 0; vv < 4; ++vv)
      *reinterpret_cast<bf16x4*>(region + tile_off64(l32, 4 * db + vv) + 8 * g32) =
          pack4(acc[db][4 * vv] * mul, acc[db][4 * vv + 1] * mul, acc[db][4 * vv + 2] * mul, acc[db][4 * vv + 3] * mul);
}
__device__ __forceinline__ void store_rows(const KArgs& a, void* out, const TStride& so, const char* region,
                                           const Run& run, int row0, int s, int b, int h, int lane) {
  const int sub = lane >> 3, ch = lane & 7;
  uint4 val[4];   // all read before the first store: a store behind a test otherwise holds up the next read
#pragma unroll
  for (int it = 0; it < 4; ++it) val[it] = *reinterpret_cast<const uint4*>(region + tile_off64(it * 8 + sub, ch));
  __bf16* head = static_cast<__bf16*>(out) + row_off(so, b, 0, h) + ch * 8;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = row0 + it * 8 + sub;
    if (row < run.len)   // not padding of a partial tile
      *reinterpret_cast<uint4*>(head + (long long)token_of(run.p0 + row, s, a.N) * so.t) = val[it];
  }
}

// ===========================================================================
// Forward: 128 query rows a workgroup, 64-key tiles, two stages (32 KB), four workgroups per CU
// (120 registers).  Bound by the vector unit (153 instructions and 16 MFMAs per 64 x 32 tile) and
// the clock it leaves.
// ===========================================================================
__global__ void __launch_bounds__(256, 4)
fwd_d64_kernel(KArgs a, int T, Deal deal, int first_block) {
  __shared__ __attribute__((aligned(1024))) char smem[4 * kTile];   // [stage][K,V]
  fetch_args(a, deal);
  const int tid = thread_id(), lane = tid & 63, w = uni(tid >> 6);
  const int g32 = lane >> 5, l32 = lane & 31;

  int seq, rank;
  if (!decode_block(first_block + block_id(), T, deal, seq, rank)) return;
  const HeadPos at = head_of_seq(a, seq);
  const int c = at.c, b = at.b, h = at.h;
  int qt = T - 1 - rank;
  const int s = uni(shift_of_head(a, h));
  Run run;
  if (!run_of_tile(a, at.g, s, kOwn, qt, run)) return;
  run.p0 = uni(run.p0); run.len = uni(run.len);
  const int i0 = uni(qt * kOwn);
  const int qw0 = i0 + 32 * w, qrow = qw0 + l32;
  const int n_tiles = uni((min(run.len, i0 + kOwn) + kTR - 1) / kTR);
  const float c2 = a.scale_log2;

  bf16x8 qf[4];
  {
    const int tok = run_token(a, run, qrow, s);
    const bf16x8* src = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(a.q) + row_off(a.sq, b, tok, h));
#pragma unroll
    for (int k = 0; k < 4; ++k) qf[k] = src[2 * k + g32];
  }
  const uint64_t k_rb = (uint64_t)a.sk.t * 2, v_rb = (uint64_t)a.sv.t * 2;
  const uint64_t k_head = uni64(reinterpret_cast<uint64_t>(a.k) + row_off(a.sk, b, 0, c) * 2);
  const uint64_t v_head = uni64(reinterpret_cast<uint64_t>(a.v) + row_off(a.sv, b, 0, c) * 2);
  const uint32_t base = lds_addr(smem);
  const Stager sg = stager(w, lane, k_rb, v_rb);
  auto issue = [&](int n, int stage) __attribute__((always_inline)) {
    stage_pair(a, run, s, n * kTR, sg, w, k_head, k_rb, v_head, v_rb, base + stage * 2 * kTile,
               base + stage * 2 * kTile + kTile);
  };

  const Offsets64 lo = lane_offsets64(lane);
  f32x16 o[2] = {zero16(), zero16()};
  float m_run = -INFINITY, l_run = 0.f;
  issue(0, 0);
  for (int n = 0; n < n_tiles; ++n) {
    const int stage = n & 1;
    wait_vmcnt0();                        // this wave's part of tile n has landed
    __syncthreads();                      // everyone's part has landed; everyone left tile n - 1
    if (n + 1 < n_tiles) issue(n + 1, stage ^ 1);
    const int j0 = n * kTR;
    const char* Ks = smem + stage * 2 * kTile;
    const char* Vs = Ks + kTile;
    if (j0 > qw0 + 31) continue;          // beyond the diagonal of this wave's rows
    f32x16 s0 = zero16(), s1 = zero16();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      s0 = mfma32(rm64<0>(Ks, lo, k), qf[k], s0);
      s1 = mfma32(rm64<32>(Ks, lo, k), qf[k], s1);
    }
    if (j0 + kTR - 1 > qw0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = j0 + 8 * (v >> 2) + 4 * g32 + (v & 3);
        if (key > qrow) s0[v] = -INFINITY;
        if (key + 32 > qrow) s1[v] = -INFINITY;
      }
    }
    // online softmax: the maximum is raised (and O rescaled) only when it grows by more than 2^8
    float ma = fmaxf(s0[0], s0[1]), mb = fmaxf(s1[0], s1[1]);
#pragma unroll
    for (int v = 2; v < 16; v += 2) {
      ma = fmaxf(fmaxf(ma, s0[v]), s0[v + 1]);
      mb = fmaxf(fmaxf(mb, s1[v]), s1[v + 1]);
    }
    const float mx = max_halves(fmaxf(ma, mb));
    if (__builtin_amdgcn_ballot_w64(mx * c2 > m_run * c2 + 8.f) != 0) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c2);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int v = 0; v < 16; ++v) { o[0][v] *= alpha; o[1][v] *= alpha; }
    }
    const float mc = m_run * c2;
    float ra = 0.f, rb = 0.f;
    bf16x8 pf[4];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      s0[v] = __builtin_amdgcn_exp2f(fmaf(s0[v], c2, -mc));
      s1[v] = __builtin_amdgcn_exp2f(fmaf(s1[v], c2, -mc));
      ra += s0[v];
      rb += s1[v];
    }
    l_run += ra + rb;
    pf[0] = pack8(s0[0], s0[1], s0[2], s0[3], s0[4], s0[5], s0[6], s0[7]);
    pf[1] = pack8(s0[8], s0[9], s0[10], s0[11], s0[12], s0[13], s0[14], s0[15]);
    pf[2] = pack8(s1[0], s1[1], s1[2], s1[3], s1[4], s1[5], s1[6], s1[7]);
    pf[3] = pack8(s1[8], s1[9], s1[10], s1[11], s1[12], s1[13], s1[14], s1[15]);
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      o[db] = mfma32(tr64<0>(Vs, lo, db), pf[0], o[db]);
      o[db] = mfma32(tr64<16>(Vs, lo, db), pf[1], o[db]);
      o[db] = mfma32(tr64<32>(Vs, lo, db), pf[2], o[db]);
      o[db] = mfma32(tr64<48>(Vs, lo, db), pf[3], o[db]);
    }
  }
  __syncthreads();
  const float l_tot = sum_halves(l_run);
  char* region = smem + w * 32 * kRow;
  wave_rows(region, o, 1.f / l_tot, l32, g32);
  __syncthreads();
  store_rows(a, a.o, a.so, region, run, qw0, s, b, h, lane);
  if (g32 == 0 && qrow < run.len)
    a.lse[((size_t)b * a.H + h) * a.N + token_of(run.p0 + qrow, s, a.N)] =
        (m_run * c2 + __builtin_amdgcn_logf(l_tot)) * kLn2;
}

// ===========================================================================
// dK/dV: 128 keys a workgroup (32 per wave), 64-row query tiles from the end of the run down to
// the diagonal, heads innermost (workgroups of one group then read the same tile at about the same
// time).  All four products in one wave: P and dS never leave its registers.  Two workgroups per
// CU.  One 32-query block after the other instead of the phases of dkdv64_tile, in one loop with the
// masked tiles: 2720 us at the size above, 2198 now.
// ===========================================================================
struct RowTerms {
  float lse2[kTR], neg_delta[kTR];
};

// One 32-query block (MB) of a tile: scores and dP - delta, and the operands made of them.
struct Block64 {
  f32x16 s, dp;
};
template <int MB>
__device__ __forceinline__ void sc_load64(bf16x8 (&buf)[8], const char* Qs, const char* dOs, const Offsets64& lo) {
#pragma unroll
  for (int k = 0; k < 4; ++k) { buf[k] = rm64<32 * MB>(Qs, lo, k); buf[4 + k] = rm64<32 * MB>(dOs, lo, k); }
}
template <int MB>
__device__ __forceinline__ void dp_init64(Block64& x, const RowTerms& rows, int g32) {
  // starts at -delta: ends as dP - delta
#pragma unroll
  for (int vv = 0; vv < 4; ++vv) {
    const float4 d4 = *reinterpret_cast<const float4*>(&rows.neg_delta[32 * MB + 8 * vv + 4 * g32]);
    x.dp[4 * vv] = d4.x; x.dp[4 * vv + 1] = d4.y; x.dp[4 * vv + 2] = d4.z; x.dp[4 * vv + 3] = d4.w;
  }
}
__device__ __forceinline__ void sc_mma64(const bf16x8 (&buf)[8], Block64& x, const bf16x8 (&kf)[4], const bf16x8 (&vf)[4]) {
  x.s = zero16();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    x.s = mfma32(buf[k], kf[k], x.s);
    x.dp = mfma32(buf[4 + k], vf[k], x.dp);
  }
}
template <int MB>
__device__ __forceinline__ void ac_load64(bf16x8 (&buf)[8], const char* Qs, const char* dOs, const Offsets64& lo) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      buf[4 * t + db] = t == 0 ? tr64<32 * MB>(dOs, lo, db) : tr64<32 * MB + 16>(dOs, lo, db);
      buf[4 * t + 2 + db] = t == 0 ? tr64<32 * MB>(Qs, lo, db) : tr64<32 * MB + 16>(Qs, lo, db);
    }
}
__device__ __forceinline__ void ac_mma64(const bf16x8 (&buf)[8], const bf16x8 (&pf)[2], const bf16x8 (&df)[2],
                                         f32x16 (&dk)[2], f32x16 (&dv)[2]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      dv[db] = mfma32(buf[4 * t + db], pf[t], dv[db]);
      dk[db] = mfma32(buf[4 * t + 2 + db], df[t], dk[db]);
    }
}
// P and dS of a block as B operands.  MASK: keys after the query, and query rows at or past q_lim
// (padding of a partial tile), give zero.
template <int MB, bool MASK>
__device__ __forceinline__ void softmax64(Block64& x, const RowTerms& rows, bf16x8 (&pf)[2], bf16x8 (&df)[2], float c2,
                                          int g32, int q_first = 0, int key = 0, int q_lim = 0) {
#pragma unroll
  for (int vv = 0; vv < 4; ++vv) {
    const float4 l4 = *reinterpret_cast<const float4*>(&rows.lse2[32 * MB + 8 * vv + 4 * g32]);
    const float ls[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int v = 4 * vv + e;
      float p = __builtin_amdgcn_exp2f(fmaf(x.s[v], c2, -ls[e]));
      if (MASK) {
        const int q = q_first + 32 * MB + 8 * vv + 4 * g32 + e;
        if (key > q || q >= q_lim) p = 0.f;
      }
      x.s[v] = p;
      x.dp[v] *= p;
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    pf[t] = pack8(x.s[8 * t], x.s[8 * t + 1], x.s[8 * t + 2], x.s[8 * t + 3], x.s[8 * t + 4], x.s[8 * t + 5],
                  x.s[8 * t + 6], x.s[8 * t + 7]);
    df[t] = pack8(x.dp[8 * t], x.dp[8 * t + 1], x.dp[8 * t + 2], x.dp[8 * t + 3], x.dp[8 * t + 4], x.dp[8 * t + 5],
                  x.dp[8 * t + 6], x.dp[8 * t + 7]);
  }
}
// A tile whose 64 query rows see all of the wave's keys, in four phases of 8 MFMAs: the vector
// work of a block sits beside the products of the other one, and every phase fetches the operands
// of the next.
__device__ __forceinline__ void dkdv64_tile(const char* Qs, const char* dOs, const RowTerms& rows, const Offsets64& lo,
                                            const bf16x8 (&kf)[4], const bf16x8 (&vf)[4], f32x16 (&dk)[2],
                                            f32x16 (&dv)[2], float c2, int g32) {
  bf16x8 fa[8], fb[8], pf0[2], df0[2], pf1[2], df1[2];
  Block64 x0, x1;
  sc_load64<0>(fa, Qs, dOs, lo);
  dp_init64<0>(x0, rows, g32);
  __builtin_amdgcn_sched_barrier(0);
  sc_load64<1>(fb, Qs, dOs, lo);
  dp_init64<1>(x1, rows, g32);
  sc_mma64(fa, x0, kf, vf);
  interleave_mfma<8, 2, 0>();
  __builtin_amdgcn_sched_barrier(0);
  ac_load64<0>(fa, Qs, dOs, lo);
  sc_mma64(fb, x1, kf, vf);
  softmax64<0, false>(x0, rows, pf0, df0, c2, g32);
  interleave_mfma<8, 3, 9>();
  __builtin_amdgcn_sched_barrier(0);
  ac_load64<1>(fb, Qs, dOs, lo);
  ac_mma64(fa, pf0, df0, dk, dv);
  softmax64<1, false>(x1, rows, pf1, df1, c2, g32);
  interleave_mfma<8, 3, 9>();
  __builtin_amdgcn_sched_barrier(0);
  ac_mma64(fb, pf1, df1, dk, dv);
  __builtin_amdgcn_sched_barrier(0);
}
// One 32-query block by itself (tiles on the diagonal, the partial last tile).
template <int MB>
__device__ __forceinline__ void dkdv64_masked(const char* Qs, const char* dOs, const RowTerms& rows, const Offsets64& lo,
                                              const bf16x8 (&kf)[4], const bf16x8 (&vf)[4], f32x16 (&dk)[2],
                                              f32x16 (&dv)[2], float c2, int g32, int q_first, int key, int q_lim) {
  bf16x8 f[8], pf[2], df[2];
  Block64 x;
  sc_load64<MB>(f, Qs, dOs, lo);
  dp_init64<MB>(x, rows, g32);
  sc_mma64(f, x, kf, vf);
  ac_load64<MB>(f, Qs, dOs, lo);
  softmax64<MB, true>(x, rows, pf, df, c2, g32, q_first, key, q_lim);
  ac_mma64(f, pf, df, dk, dv);
}

// smem: [stage][Q,dO]
__device__ __forceinline__ void dkdv64_workgroup(const KArgs& a, int T, const Deal& deal, int block, int tid, char* smem,
                                                 RowTerms (&rows_s)[2]) {
  const int lane = tid & 63, w = uni(tid >> 6);
  const int g32 = lane >> 5, l32 = lane & 31;

  int seq, jt;
  if (!decode_block(block, T, deal, seq, jt)) return;
  const KvPos at = kv_of_seq(a, seq);
  const int c = at.c, b = at.b;
  int h_lo, nheads, s;
  part_heads(a, c, at.part, h_lo, nheads, s);
  s = uni(s);
  Run run;
  if (!run_of_tile(a, at.g, s, kOwn, jt, run)) return;
  run.p0 = uni(run.p0); run.len = uni(run.len);
  const int j0 = uni(jt * kOwn);
  const int kw0 = j0 + 32 * w, key = kw0 + l32;
  const int nq = uni((run.len - j0 + kTR - 1) / kTR);   // query tiles of one head
  const int n_iter = nheads * nq;
  const float c2 = a.scale_log2;

  bf16x8 kf[4], vf[4];   // K^T and V^T of this wave's keys
  {
    const int tok = run_token(a, run, key, s);
    const bf16x8* ks = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(a.k) + row_off(a.sk, b, tok, c));
    const bf16x8* vs = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(a.v) + row_off(a.sv, b, tok, c));
#pragma unroll
    for (int k = 0; k < 4; ++k) { kf[k] = ks[2 * k + g32]; vf[k] = vs[2 * k + g32]; }
  }
  const uint64_t q_rb = (uint64_t)a.sq.t * 2, do_rb = (uint64_t)a.so.t * 2;
  const uint64_t q_batch = uni64(reinterpret_cast<uint64_t>(a.q) + row_off(a.sq, b, 0, 0) * 2);
  const uint64_t do_batch = uni64(reinterpret_cast<uint64_t>(a.dout) + row_off(a.so, b, 0, 0) * 2);
  const uint32_t base = lds_addr(smem), rows_base = lds_addr(rows_s);
  const Stager sg = stager(w, lane, q_rb, do_rb);
  auto issue = [&](int hh, int it, int stage) __attribute__((always_inline)) {
    const int h = h_lo + hh, t0 = j0 + it * kTR;
    stage_pair(a, run, s, t0, sg, w, q_batch + (uint64_t)h * a.sq.h * 2, q_rb, do_batch + (uint64_t)h * a.so.h * 2,
               do_rb, base + stage * 2 * kTile, base + stage * 2 * kTile + kTile);
    if (w < 2) {   // wave 0: lse * log2(e), wave 1: -delta
      const float* src = (w == 0 ? a.lse2 : a.neg_delta) + ((size_t)b * a.H + h) * a.N + run_token(a, run, t0 + lane, s);
      dma4(src, rows_base + stage * (uint32_t)sizeof(RowTerms) + w * kTR * 4);
    }
  };

  const Offsets64 lo = lane_offsets64(lane);
  f32x16 dk[2] = {zero16(), zero16()}, dv[2] = {zero16(), zero16()};
  // Waits for tile n of the walk (query tile it of head hh, in stage n mod 2) and starts the
  // staging of the next one: the next head of the same query tile, else the first of the one before.
  auto begin_tile = [&](int n, int hh, int it) __attribute__((always_inline)) {
    wait_vmcnt0();
    __syncthreads();
    if (n + 1 < n_iter) {
      const bool wrap = hh + 1 == nheads;
      issue(wrap ? 0 : hh + 1, wrap ? it - 1 : it, (n & 1) ^ 1);
    }
    __builtin_amdgcn_sched_barrier(0);   // keeps the addresses out of the tile body
  };
  if (n_iter > 0) issue(0, nq - 1, 0);   // (a part may be empty)
  // the interior tiles have a loop of their own (a loop with both kinds of tile moves all
  // accumulators twice per tile); the partial last tile comes before, those on the diagonal after
  int n = 0;
  auto masked_tiles = [&](int it) __attribute__((always_inline)) {
    const int q0 = j0 + it * kTR;
    for (int hh = 0; hh < nheads; ++hh, ++n) {
      begin_tile(n, hh, it);
      const char* Qs = smem + (n & 1) * 2 * kTile;
      // blocks before this wave's keys see none of them; rows >= run.len are padding
      if (q0 + 31 >= kw0)
        dkdv64_masked<0>(Qs, Qs + kTile, rows_s[n & 1], lo, kf, vf, dk, dv, c2, g32, q0, key, run.len);
      if (q0 + 63 >= kw0)
        dkdv64_masked<1>(Qs, Qs + kTile, rows_s[n & 1], lo, kf, vf, dk, dv, c2, g32, q0, key, run.len);
    }
  };
  int it = nq - 1;
  if (run.len % kTR != 0 && it >= 2) masked_tiles(it--);
  for (; it >= 2; --it)
    for (int hh = 0; hh < nheads; ++hh, ++n) {
      begin_tile(n, hh, it);
      const char* Qs = smem + (n & 1) * 2 * kTile;
      dkdv64_tile(Qs, Qs + kTile, rows_s[n & 1], lo, kf, vf, dk, dv, c2, g32);
    }
  for (; it >= 0; --it) masked_tiles(it);
  __syncthreads();

  if (a.dkv_partial) {   // query heads cut into parts: fp32 partial of this one, summed by the combine pass
    if (key >= run.len) return;
    const size_t elems = (size_t)a.B * a.N * a.Hkv * DH;
    const int tok = token_of(run.p0 + key, s, a.N);
    float* dk_out = a.dkv_partial + (size_t)at.part * elems + ((size_t)((size_t)b * a.N + tok) * a.Hkv + c) * DH + 4 * g32;
    float* dv_out = dk_out + (size_t)a.parts * elems;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int vv = 0; vv < 4; ++vv) {
        *reinterpret_cast<float4*>(dk_out + 32 * db + 8 * vv) = make_float4(
            dk[db][4 * vv] * a.scale, dk[db][4 * vv + 1] * a.scale, dk[db][4 * vv + 2] * a.scale, dk[db][4 * vv + 3] * a.scale);
        *reinterpret_cast<float4*>(dv_out + 32 * db + 8 * vv) =
            make_float4(dv[db][4 * vv], dv[db][4 * vv + 1], dv[db][4 * vv + 2], dv[db][4 * vv + 3]);
      }
    return;
  }
  char* rk = smem + w * 32 * kRow;
  char* rv = smem + (4 + w) * 32 * kRow;
  wave_rows(rk, dk, a.scale, l32, g32);
  wave_rows(rv, dv, 1.f, l32, g32);
  __syncthreads();
  store_rows(a, a.dk, a.sdk, rk, run, kw0, s, b, c, lane);
  store_rows(a, a.dv, a.sdv, rv, run, kw0, s, b, c, lane);
}

// ===========================================================================
// dQ: 128 query rows a workgroup (32 per wave), 64-key tiles up to the diagonal, S and dP
// recomputed.  Three workgroups per CU (156 registers).
// ===========================================================================
template <int ROW0>
__device__ __forceinline__ void dq64_block(const char* Ks, const char* Vs, const Offsets64& lo, const bf16x8 (&qf)[4],
                                           const bf16x8 (&dof)[4], const f32x16& neg_delta, f32x16 (&dq)[2], float c2,
                                           float lse2, int j0, int qrow, int g32, bool masked) {
  f32x16 sx = zero16(), dp = neg_delta;   // dP - delta
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    sx = mfma32(rm64<ROW0>(Ks, lo, k), qf[k], sx);
    dp = mfma32(rm64<ROW0>(Vs, lo, k), dof[k], dp);
  }
  if (masked) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (j0 + ROW0 + 8 * (v >> 2) + 4 * g32 + (v & 3) > qrow) sx[v] = -INFINITY;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) dp[v] *= __builtin_amdgcn_exp2f(fmaf(sx[v], c2, -lse2));
  const bf16x8 d0 = pack8(dp[0], dp[1], dp[2], dp[3], dp[4], dp[5], dp[6], dp[7]);
  const bf16x8 d1 = pack8(dp[8], dp[9], dp[10], dp[11], dp[12], dp[13], dp[14], dp[15]);
#pragma unroll
  for (int db = 0; db < 2; ++db) {
    dq[db] = mfma32(tr64<ROW0>(Ks, lo, db), d0, dq[db]);
    dq[db] = mfma32(tr64<ROW0 + 16>(Ks, lo, db), d1, dq[db]);
  }
}

// smem: [stage][K,V]
__device__ __forceinline__ void dq64_workgroup(const KArgs& a, int T, const Deal& deal, int block, int tid, char* smem) {
  const int lane = tid & 63, w = uni(tid >> 6);
  const int g32 = lane >> 5, l32 = lane & 31;

  int seq, rank;
  if (!decode_block(block, T, deal, seq, rank)) return;
  const HeadPos at = head_of_seq(a, seq);
  const int c = at.c, b = at.b, h = at.h;
  int qt = T - 1 - rank;
  const int s = uni(shift_of_head(a, h));
  Run run;
  if (!run_of_tile(a, at.g, s, kOwn, qt, run)) return;
  run.p0 = uni(run.p0); run.len = uni(run.len);
  const int i0 = uni(qt * kOwn);
  const int qw0 = i0 + 32 * w, qrow = qw0 + l32;
  const int n_tiles = uni((min(run.len, i0 + kOwn) + kTR - 1) / kTR);
  const float c2 = a.scale_log2;

  bf16x8 qf[4], dof[4];
  f32x16 neg_delta;
  float lse2;
  {
    const int tok = run_token(a, run, qrow, s);
    const bf16x8* qs = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(a.q) + row_off(a.sq, b, tok, h));
    const bf16x8* ds = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(a.dout) + row_off(a.so, b, tok, h));
#pragma unroll
    for (int k = 0; k < 4; ++k) { qf[k] = qs[2 * k + g32]; dof[k] = ds[2 * k + g32]; }
    const size_t ro = ((size_t)b * a.H + h) * a.N + tok;
    lse2 = a.lse2[ro];
    const float nd = a.neg_delta[ro];
#pragma unroll
    for (int v = 0; v < 16; ++v) neg_delta[v] = nd;
  }
  const uint64_t k_rb = (uint64_t)a.sk.t * 2, v_rb = (uint64_t)a.sv.t * 2;
  const uint64_t k_head = uni64(reinterpret_cast<uint64_t>(a.k) + row_off(a.sk, b, 0, c) * 2);
  const uint64_t v_head = uni64(reinterpret_cast<uint64_t>(a.v) + row_off(a.sv, b, 0, c) * 2);
  const uint32_t base = lds_addr(smem);
  const Stager sg = stager(w, lane, k_rb, v_rb);
  auto issue = [&](int n, int stage) __attribute__((always_inline)) {
    stage_pair(a, run, s, n * kTR, sg, w, k_head, k_rb, v_head, v_rb, base + stage * 2 * kTile,
               base + stage * 2 * kTile + kTile);
  };

  const Offsets64 lo = lane_offsets64(lane);
  f32x16 dq[2] = {zero16(), zero16()};
  issue(0, 0);
  for (int n = 0; n < n_tiles; ++n) {
    const int stage = n & 1;
    wait_vmcnt0();
    __syncthreads();
    if (n + 1 < n_tiles) issue(n + 1, stage ^ 1);
    const int j0 = n * kTR;
    const char* Ks = smem + stage * 2 * kTile;
    const char* Vs = Ks + kTile;
    if (j0 > qw0 + 31) continue;
    const bool masked = j0 + kTR - 1 > qw0;
    dq64_block<0>(Ks, Vs, lo, qf, dof, neg_delta, dq, c2, lse2, j0, qrow, g32, masked);
    dq64_block<32>(Ks, Vs, lo, qf, dof, neg_delta, dq, c2, lse2, j0, qrow, g32, masked);
  }
  __syncthreads();
  char* region = smem + w * 32 * kRow;
  wave_rows(region, dq, a.scale, l32, g32);
  __syncthreads();
  store_rows(a, a.dq, a.sdq, region, run, qw0, s, b, h, lane);
}

__global__ void __launch_bounds__(256, 2)
bwd_dkdv_d64_kernel(KArgs a, int T, Deal deal, int first_block) {
  __shared__ __attribute__((aligned(1024))) char smem[4 * kTile];
  __shared__ __attribute__((aligned(1024))) RowTerms rows_s[2];
  dkdv64_workgroup(a, T, deal, first_block + block_id(), thread_id(), smem, rows_s);
}

__global__ void __launch_bounds__(256, 3)
bwd_dq_d64_kernel(KArgs a, int T, Deal deal, int first_block) {
  __shared__ __attribute__((aligned(1024))) char smem[4 * kTile];
  dq64_workgroup(a, T, deal, first_block + block_id(), thread_id(), smem);
}

// Both in one launch, dK/dV first: neither needs the other, and where they do not fill the chip their
// chains of tiles run side by side.
__global__ void __launch_bounds__(256, 2)
bwd_both_d64_kernel(KArgs a, int n_kv, int T, Deal deal_kv, Deal deal_q) {
  __shared__ __attribute__((aligned(1024))) char smem[4 * kTile];
  __shared__ __attribute__((aligned(1024))) RowTerms rows_s[2];
  if (block_id() < n_kv)
    dkdv64_workgroup(a, T, deal_kv, block_id(), thread_id(), smem, rows_s);
  else
    dq64_workgroup(a, T, deal_q, block_id() - n_kv, thread_id(), smem);
}

}  // namespace

int launch_fwd_d64(const KArgs& a, hipStream_t st) {
  const int T = ragged_tiles(a, kOwn);
  const Grid g = grid_of(T, a.B * a.H * a.NG, a.r, 128);   // 32 CUs per XCD, four workgroups each
  return launch_blocks(fwd_d64_kernel, g.blocks, 256, st, a, T, g.deal);
}

int launch_bwd_dkdv_d64(const KArgs& a, hipStream_t st) {
  const int T = ragged_tiles(a, kOwn);
  const Grid g = grid_of(T, a.B * a.Hkv * a.NG * a.parts, 1, 64);
  return launch_blocks(bwd_dkdv_d64_kernel, g.blocks, 256, st, a, T, g.deal);
}

// dK/dV and dQ in one launch, dK/dV first; 1 and no launch where one by one is better.  Up to twenty
// workgroups per CU, ten rounds of two: dQ fills the tail of dK/dV, whose workgroups are few and
// uneven with several query heads to a kv head.  Forward + backward, one by one and in one launch:
// N = 1024, H = 4, Hkv = 2 34.7 and 26.4 us; N = 8192, H = 32, Hkv = 32 / 1 377 / 413 and 364 / 357;
// N = 8192, H = 64, Hkv = 8 (4608 workgroups) 801 and 698.  Beyond, dQ's third workgroup on a CU is
// worth more: N = 16384, H = 32 (8192 workgroups) 1398 and 1406.  dQ first: 242 us where dK/dV first
// takes 205 and one by one 229 (B = 2, N = 4096, H = 32, Hkv = 8), at best even elsewhere.
int launch_bwd_both_d64(const KArgs& a, hipStream_t st) {
  const int T = ragged_tiles(a, kOwn);
  const Grid kv = grid_of(T, a.B * a.Hkv * a.NG * a.parts, 1, 64), q = grid_of(T, a.B * a.H * a.NG, a.r, 64);
  if (kv.blocks + q.blocks > kOneLaunchBlocks64) return 1;
  hipLaunchKernelGGL(bwd_both_d64_kernel, dim3(kv.blocks + q.blocks), dim3(256), 0, st, a,
                     kv.blocks, T, kv.deal, q.deal);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_bwd_dq_d64(const KArgs& a, hipStream_t st) {
  const int T = ragged_tiles(a, kOwn);
  const Grid g = grid_of(T, a.B * a.H * a.NG, a.r, 96);
  return launch_blocks(bwd_dq_d64_kernel, g.blocks, 256, st, a, T, g.deal);
}

}  // namespace s2
