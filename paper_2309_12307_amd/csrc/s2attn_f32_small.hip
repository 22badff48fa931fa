// fp32 S2-Attn kernels (forward; backward) for problems of few rows: the same instruction, operand
// layout and arithmetic as s2attn_f32.hip, dealt out finer.
//
// What bounds a small problem is the chain of tiles of one workgroup while most of the chip is idle.
// Here a workgroup owns 16 rows and its four waves share out the tiles of 16 rows that these meet, so
// there are four times the workgroups and a quarter of the chain.  A tile then serves one wave only, and
// both operand forms (16 rows of a column of chunks; 4 rows of 64 columns) are whole 64- and 256-byte
// pieces of memory, so they go straight from global memory to registers: no LDS, no barrier, and an
// operand's registers are loaded for the next tile as soon as this tile's products have been issued.
// The waves' sums meet in LDS once, at the end.
//
// Forward and backward, us, 64 rows to a workgroup and here: N = 256, H = 4, D = 64, G = 64: 6.4 + 9.3 and
// 4.7 + 7.1; N = 1000, H = 4, Hkv = 2, D = 128, G = 500: 44.7 + 85.0 and 16.7 + 62.0; N = 1024, H = 8, D = 64,
// G = 1024: 53.8 + 92.7 and 23.1 + 64.0.  The backward reads a tile in five forms (40 KB for 4096 MFMA cycles
// of four waves at D = 128), which is what the caches give once the CUs of an XCD have their workgroups (whole sequences go
// to an XCD, so one sequence keeps to 32 CUs): the lines at small_fwd and small_bwd lie there, and at the length
// from which the tiles in LDS feed a chain better.  Two waves to a tile (32 rows to a workgroup) is not faster anywhere
// but between 128 and 256 workgroups of 64 rows (5 %).
#include <cfloat>

#include "s2attn_f32_common.h"
#include "s2attn_launch.h"

namespace s2 {
namespace {

constexpr int kRows = 16;     // rows of a workgroup, and of a tile
constexpr int kWaves = 4;

// Row-major operand: X[row][16 i + 4 q4 ..], `row` this lane's (c16) row.
template <int D>
__device__ __forceinline__ void load_rm(f32x4 (&x)[D / 16], const float* row, int q4) {
#pragma unroll
  for (int i = 0; i < D / 16; ++i) x[i] = *reinterpret_cast<const f32x4*>(row + 16 * i + 4 * q4);
}

// Transposed operand: X[4 q4 + v][64 j + 4 c16 ..], rows of the tile that starts at row i0 of the run.
template <int D>
__device__ __forceinline__ void load_tr(f32x4 (&x)[4][D / 64], const KArgs& a, const void* src, const TStride& st, const Run& run,
                                        int s, int b, int head, int i0, int c16, int q4) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const float* row = static_cast<const float*>(src) + row_off(st, b, run_token(a, run, i0 + 4 * q4 + v, s), head);
#pragma unroll
    for (int j = 0; j < D / 64; ++j) x[v][j] = *reinterpret_cast<const f32x4*>(row + 64 * j + 4 * c16);
  }
}

// acc += X own^T over D, in two chains
template <int D>
__device__ __forceinline__ f32x4 scores(const f32x4 (&x)[D / 16], const f32x4 (&own)[D / 16], f32x4 acc) {
  f32x4 odd = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < D / 16; i += 2)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc = mfma4(x[i][e], own[i][e], acc);
      odd = mfma4(x[i + 1][e], own[i + 1][e], odd);
    }
  return acc + odd;
}

template <int D>
__device__ __forceinline__ void accumulate(f32x4 (&acc)[D / 64][4], const f32x4 (&x)[4][D / 64], f32x4 wt) {
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int j = 0; j < D / 64; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j][e] = mfma4(x[v][j][e], wt[v], acc[j][e]);
}

template <int D>
__device__ __forceinline__ void zero(f32x4 (&acc)[D / 64][4]) {
#pragma unroll
  for (int j = 0; j < D / 64; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[j][e] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// A wave's 16 x D block in LDS, one row to a lane of the accumulators; rows four floats longer than D so
// that the 16 rows do not start at one bank.
template <int D>
constexpr int kBlockFloats = kRows * (D + 4);

// Reads float4 `f` (0 .. 4 D - 1) of the sum of the waves' blocks, each times its factor.
template <int D>
__device__ __forceinline__ f32x4 sum_blocks(const float* blocks, int f, const float (&factor)[kWaves]) {
  const int row = f / (D / 4), col = f % (D / 4);
  f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < kWaves; ++w)
    x += *reinterpret_cast<const f32x4*>(blocks + w * kBlockFloats<D> + row * (D + 4) + 4 * col) * factor[w];
  return x;
}

template <int D>
__global__ void __launch_bounds__(64 * kWaves, 2) fwd_f32_small_kernel(KArgs a, int T, Deal deal, int first_block) {
  __shared__ __attribute__((aligned(16))) float blocks[kWaves * kBlockFloats<D>];
  __shared__ float max_s[kWaves][kRows], sum_s[kWaves][kRows];
  fetch_args(a, deal);

  const int tid = thread_id(), lane = tid & 63, w = uni(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  int seq, rank;
  if (!decode_block(first_block + block_id(), T, deal, seq, rank)) return;
  const HeadPos at = head_of_seq(a, seq);
  const int s = uni(shift_of_head(a, at.h));
  Run run;
  int qt = T - 1 - rank;
  if (!run_of_tile(a, at.g, s, kRows, qt, run)) return;
  run.p0 = uni(run.p0); run.len = uni(run.len);
  const int i0 = uni(qt * kRows), qrow = i0 + c16;
  const int tok = run_token(a, run, qrow, s);
  const float c2 = a.scale_log2;

  f32x4 qf[D / 16], kf[D / 16], vf[4][D / 64], o[D / 64][4];
  auto load_k = [&](int jt) __attribute__((always_inline)) {
    load_rm<D>(kf, static_cast<const float*>(a.k) + row_off(a.sk, at.b, run_token(a, run, jt * kRows + c16, s), at.c), q4);
  };
  auto load_v = [&](int jt) __attribute__((always_inline)) {
    load_tr<D>(vf, a, a.v, a.sv, run, s, at.b, at.c, jt * kRows, c16, q4);
  };
  const int last = i0 / kRows;   // the tile on the diagonal
  if (w <= last) {
    load_k(w);
    load_rm<D>(qf, static_cast<const float*>(a.q) + row_off(a.sq, at.b, tok, at.h), q4);
    load_v(w);
  }
  zero<D>(o);
  float m_run = -FLT_MAX, l_run = 0.f;   // as in fwd_f32_kernel
  for (int jt = w; jt <= last; jt += kWaves) {
    const bool more = jt + kWaves <= last;
    f32x4 sc = scores<D>(kf, qf, f32x4{0.f, 0.f, 0.f, 0.f});
    if (more) load_k(jt + kWaves);
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      sc[v] *= c2;
      if (jt == last && 4 * q4 + v > c16) sc[v] = -INFINITY;
      mx = fmaxf(mx, sc[v]);
    }
    mx = max_cols(mx);
    if (__builtin_amdgcn_ballot_w64(mx > m_run) != 0) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int j = 0; j < D / 64; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[j][e] *= alpha;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      sc[v] = exp2f(sc[v] - m_run);
      l_run += sc[v];
    }
    accumulate<D>(o, vf, sc);
    if (more) load_v(jt + kWaves);
  }
  l_run = sum_cols(l_run);
  store_row<D>(blocks + w * kBlockFloats<D> + c16 * (D + 4), o, 1.f, q4);
  if (q4 == 0) {
    max_s[w][c16] = m_run;
    sum_s[w][c16] = l_run;
  }
  __syncthreads();

#pragma unroll
  for (int f = tid; f < kRows * D / 4; f += 64 * kWaves) {
    const int row = f / (D / 4);
    if (i0 + row >= run.len) break;
    float m = max_s[0][row], factor[kWaves], l = 0.f;
#pragma unroll
    for (int x = 1; x < kWaves; ++x) m = fmaxf(m, max_s[x][row]);
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      factor[x] = exp2f(max_s[x][row] - m);
      l = fmaf(sum_s[x][row], factor[x], l);
    }
    const f32x4 r = sum_blocks<D>(blocks, f, factor) * (1.f / l);
    const int t = token_of(run.p0 + i0 + row, s, a.N);
    *reinterpret_cast<f32x4*>(static_cast<float*>(a.o) + row_off(a.so, at.b, t, at.h) + 4 * (f % (D / 4))) = r;
    if (f % (D / 4) == 0) a.lse[((size_t)at.b * a.H + at.h) * a.N + t] = (m + log2f(l)) * kLn2;
  }
}

// ---------------------------------------------------------------------------
// Backward, one launch as in bwd_f32_kernel.  dK/dV: 16 keys; the waves share out the tiles of 16 query
// rows, all query heads of the part.  dQ: 16 query rows; the waves share out the key tiles.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void dkdv_small_block(const KArgs& a, float* blocks, int block, int T, const Deal& deal) {
  const int tid = thread_id(), lane = tid & 63, w = uni(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  int seq, kt;
  if (!decode_block(block, T, deal, seq, kt)) return;
  const KvPos at = kv_of_seq(a, seq);
  int h_lo, nheads, s;
  part_heads(a, at.c, at.part, h_lo, nheads, s);
  Run run;
  if (!run_of_tile(a, at.g, s, kRows, kt, run)) return;
  run.p0 = uni(run.p0); run.len = uni(run.len);
  const int j0 = uni(kt * kRows), key = j0 + c16;
  const int nq = uni((run.len - 1) / kRows) - j0 / kRows + 1;   // query tiles of a head, from the diagonal on
  const float c2 = a.scale_log2;

  const int tok = run_token(a, run, j0 + c16, s);
  f32x4 kf[D / 16], vf[D / 16], qf[D / 16], gf[D / 16], of[D / 16], qt[4][D / 64], gt[4][D / 64], dk[D / 64][4], dv[D / 64][4];
  float lse = 0.f;
  // first row of the it-th query tile: from the end of the run to the diagonal, so that the large
  // probabilities are added last
  auto first_row = [&](int it) __attribute__((always_inline)) { return j0 + (nq - 1 - it) * kRows; };
  auto load_rows = [&](int h, int it) __attribute__((always_inline)) {
    const int t = run_token(a, run, first_row(it) + c16, s);
    load_rm<D>(qf, static_cast<const float*>(a.q) + row_off(a.sq, at.b, t, h), q4);
    load_rm<D>(gf, static_cast<const float*>(a.dout) + row_off(a.so, at.b, t, h), q4);
    load_rm<D>(of, static_cast<const float*>(a.o) + row_off(a.so, at.b, t, h), q4);
    lse = a.lse[((size_t)at.b * a.H + h) * a.N + t];
  };
  auto load_gt = [&](int h, int it) __attribute__((always_inline)) {
    load_tr<D>(gt, a, a.dout, a.so, run, s, at.b, h, first_row(it), c16, q4);
  };
  auto load_qt = [&](int h, int it) __attribute__((always_inline)) {
    load_tr<D>(qt, a, a.q, a.sq, run, s, at.b, h, first_row(it), c16, q4);
  };
  zero<D>(dk);
  zero<D>(dv);
  // the wave's share of the tiles (head h_lo + hh, query tile it)
  int hh = 0, it = w;
  auto settle = [&](int& x, int& y) __attribute__((always_inline)) {
    while (x < nheads && y >= nq) { y -= nq; ++x; }
  };
  settle(hh, it);
  if (hh < nheads) {
    load_rm<D>(kf, static_cast<const float*>(a.k) + row_off(a.sk, at.b, tok, at.c), q4);
    load_rm<D>(vf, static_cast<const float*>(a.v) + row_off(a.sv, at.b, tok, at.c), q4);
    if constexpr (D == 64) {
      load_rows(h_lo + hh, it);
      load_gt(h_lo + hh, it);
      load_qt(h_lo + hh, it);
    }
  }
  // D = 64: an operand is loaded for the next tile once this tile's products are out; D = 128 has no
  // registers left for that and loads a tile's operands together.
  while (hh < nheads) {
    const int q0 = first_row(it);
    int hn = hh, in = it + kWaves;
    settle(hn, in);
    const bool more = hn < nheads;
    if constexpr (D == 128) {
      load_rows(h_lo + hh, it);
      load_gt(h_lo + hh, it);
      load_qt(h_lo + hh, it);
    }
    f32x4 sc = scores<D>(qf, kf, f32x4{0.f, 0.f, 0.f, 0.f});
    f32x4 dp = scores<D>(gf, vf, f32x4{0.f, 0.f, 0.f, 0.f});
    f32x4 part = of[0] * gf[0];
#pragma unroll
    for (int i = 1; i < D / 16; ++i) part += of[i] * gf[i];
    const float delta = sum_cols((part[0] + part[1]) + (part[2] + part[3]));
    const float l = lse * kLog2e;
    if (D == 64 && more) load_rows(h_lo + hn, in);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = q0 + 4 * q4 + v;
      float p = exp2f(fmaf(sc[v], c2, -__shfl(l, 4 * q4 + v)));
      if (key > i || i >= run.len) p = 0.f;
      sc[v] = p;
      dp[v] = (dp[v] - __shfl(delta, 4 * q4 + v)) * p;
    }
    accumulate<D>(dv, gt, sc);
    if (D == 64 && more) load_gt(h_lo + hn, in);
    accumulate<D>(dk, qt, dp);
    if (D == 64 && more) load_qt(h_lo + hn, in);
    hh = hn;
    it = in;
  }

  float* dv_blocks = blocks + kWaves * kBlockFloats<D>;
  store_row<D>(blocks + w * kBlockFloats<D> + c16 * (D + 4), dk, a.scale, q4);
  store_row<D>(dv_blocks + w * kBlockFloats<D> + c16 * (D + 4), dv, 1.f, q4);
  __syncthreads();
  float one[kWaves];
#pragma unroll
  for (int x = 0; x < kWaves; ++x) one[x] = 1.f;
  const size_t elems = (size_t)a.B * a.N * a.Hkv * D;
#pragma unroll
  for (int f = tid; f < kRows * D / 4; f += 64 * kWaves) {
    const int row = f / (D / 4), col = 4 * (f % (D / 4));
    if (j0 + row >= run.len) break;
    const int t = token_of(run.p0 + j0 + row, s, a.N);
    const f32x4 x = sum_blocks<D>(blocks, f, one), y = sum_blocks<D>(dv_blocks, f, one);
    if (a.dkv_partial) {   // contiguous fp32 partial of this part, summed by the combine pass
      float* dst = a.dkv_partial + at.part * elems + ((size_t)((size_t)at.b * a.N + t) * a.Hkv + at.c) * D + col;
      *reinterpret_cast<f32x4*>(dst) = x;
      *reinterpret_cast<f32x4*>(dst + a.parts * elems) = y;
    } else {
      *reinterpret_cast<f32x4*>(static_cast<float*>(a.dk) + row_off(a.sdk, at.b, t, at.c) + col) = x;
      *reinterpret_cast<f32x4*>(static_cast<float*>(a.dv) + row_off(a.sdv, at.b, t, at.c) + col) = y;
    }
  }
}

template <int D>
__device__ __forceinline__ void dq_small_block(const KArgs& a, float* blocks, int block, int T, const Deal& deal) {
  const int tid = thread_id(), lane = tid & 63, w = uni(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  int seq, rank;
  if (!decode_block(block, T, deal, seq, rank)) return;
  const HeadPos at = head_of_seq(a, seq);
  const int s = uni(shift_of_head(a, at.h));
  Run run;
  int qt = T - 1 - rank;
  if (!run_of_tile(a, at.g, s, kRows, qt, run)) return;
  run.p0 = uni(run.p0); run.len = uni(run.len);
  const int i0 = uni(qt * kRows), qrow = i0 + c16;
  const int tok = run_token(a, run, qrow, s);
  const float c2 = a.scale_log2;

  f32x4 qf[D / 16], gf[D / 16], kf[D / 16], vf[D / 16], kt[4][D / 64], dq[D / 64][4];
  auto load_k = [&](int jt) __attribute__((always_inline)) {
    load_rm<D>(kf, static_cast<const float*>(a.k) + row_off(a.sk, at.b, run_token(a, run, jt * kRows + c16, s), at.c), q4);
  };
  auto load_v = [&](int jt) __attribute__((always_inline)) {
    load_rm<D>(vf, static_cast<const float*>(a.v) + row_off(a.sv, at.b, run_token(a, run, jt * kRows + c16, s), at.c), q4);
  };
  auto load_kt = [&](int jt) __attribute__((always_inline)) {
    load_tr<D>(kt, a, a.k, a.sk, run, s, at.b, at.c, jt * kRows, c16, q4);
  };
  const int last = i0 / kRows;
  float delta = 0.f, lse2 = 0.f;
  if (w <= last) {
    load_k(w);
    load_rm<D>(qf, static_cast<const float*>(a.q) + row_off(a.sq, at.b, tok, at.h), q4);
    load_v(w);
    load_rm<D>(gf, static_cast<const float*>(a.dout) + row_off(a.so, at.b, tok, at.h), q4);
    f32x4 of[D / 16];
    load_rm<D>(of, static_cast<const float*>(a.o) + row_off(a.so, at.b, tok, at.h), q4);
    lse2 = a.lse[((size_t)at.b * a.H + at.h) * a.N + tok] * kLog2e;
    load_kt(w);
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) delta = fmaf(of[i][e], gf[i][e], delta);
    delta = sum_cols(delta);
  }
  zero<D>(dq);
  for (int jt = w; jt <= last; jt += kWaves) {
    const bool more = jt + kWaves <= last;
    f32x4 sc = scores<D>(kf, qf, f32x4{0.f, 0.f, 0.f, 0.f});
    if (more) load_k(jt + kWaves);
    f32x4 dp = scores<D>(vf, gf, f32x4{-delta, -delta, -delta, -delta});
    if (more) load_v(jt + kWaves);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float p = exp2f(fmaf(sc[v], c2, -lse2));
      if (jt == last && 4 * q4 + v > c16) p = 0.f;
      dp[v] *= p;
    }
    accumulate<D>(dq, kt, dp);
    if (more) load_kt(jt + kWaves);
  }
  store_row<D>(blocks + w * kBlockFloats<D> + c16 * (D + 4), dq, a.scale, q4);
  __syncthreads();
  float one[kWaves];
#pragma unroll
  for (int x = 0; x < kWaves; ++x) one[x] = 1.f;
#pragma unroll
  for (int f = tid; f < kRows * D / 4; f += 64 * kWaves) {
    const int row = f / (D / 4);
    if (i0 + row >= run.len) break;
    const int t = token_of(run.p0 + i0 + row, s, a.N);
    *reinterpret_cast<f32x4*>(static_cast<float*>(a.dq) + row_off(a.sdq, at.b, t, at.h) + 4 * (f % (D / 4))) =
        sum_blocks<D>(blocks, f, one);
  }
}

template <int D>
__global__ void __launch_bounds__(64 * kWaves, 2)
bwd_f32_small_kernel(KArgs a, int n_kv, int T, Deal deal_kv, Deal deal_q, int first_block) {
  __shared__ __attribute__((aligned(16))) float blocks[2 * kWaves * kBlockFloats<D>];
  fetch_args(a, deal_q);
  const int block = first_block + block_id();
  if (block < n_kv)
    dkdv_small_block<D>(a, blocks, block, T, deal_kv);
  else
    dq_small_block<D>(a, blocks, block - n_kv, T, deal_q);
}

template <int D>
int launch_fwd_t(const KArgs& a, hipStream_t st) {
  const int T = ragged_tiles(a, kRows);
  const Grid g = grid_of(T, a.B * a.H * a.NG, a.r, 64);
  return launch_blocks(fwd_f32_small_kernel<D>, g.blocks, 64 * kWaves, st, a, T, g.deal);
}

template <int D>
int launch_bwd_t(const KArgs& a, bool dq_last, hipStream_t st) {
  const int T = ragged_tiles(a, kRows);
  const Grid kv = grid_of(T, a.B * a.Hkv * a.NG * a.parts, 1, 64), q = grid_of(T, a.B * a.H * a.NG, a.r, 64);
  const int n_first = dq_last ? kv.blocks : kv.blocks + q.blocks;
  const int rc = launch_blocks(bwd_f32_small_kernel<D>, n_first, 64 * kWaves, st, a, kv.blocks, T, kv.deal, q.deal);
  if (rc != 0 || !dq_last) return rc;
  return launch_blocks(bwd_f32_small_kernel<D>, q.blocks, 64 * kWaves, st, a, 0, T, kv.deal, q.deal);
}

}  // namespace

int launch_fwd_f32_small(const KArgs& a, hipStream_t st) {
  return a.D == 64 ? launch_fwd_t<64>(a, st) : launch_fwd_t<128>(a, st);
}

int launch_bwd_f32_small(const KArgs& a, bool dq_last, hipStream_t st) {
  return a.D == 64 ? launch_bwd_t<64>(a, dq_last, st) : launch_bwd_t<128>(a, dq_last, st);
}

}  // namespace s2
