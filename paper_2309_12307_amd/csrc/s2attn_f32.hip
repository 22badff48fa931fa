// fp32 S2-Attn kernels (forward; backward) for gfx950 on the fp32 matrix instruction
// v_mfma_f32_16x16x4_f32: fp32 operands, fp32 products and sums, twice the rate of the vector
// unit's fp32 fma.  Any even group size and any shift (partial tiles are masked); the shift and
// the grouping of LongLoRA Algorithm 1 are row-address arithmetic only (run_token).
//
// What bounds them: the matrix unit (256 flop per clock and CU).  An instruction takes 32
// cycles, so LDS traffic, the softmax and the staging are all small beside it, and the layout
// is chosen for few instructions per MFMA: every LDS operand is a 16-byte read that feeds four
// MFMAs, and no accumulator is ever moved between lanes.
//
// Lane l: c16 = l % 16, q4 = l / 16.  Operand layout of the instruction: A row c16, B column
// c16, contraction slot q4; C column c16, register v holds row 4 q4 + v.
//   row-major operand (contraction over d): a lane reads X[row c16][16 i + 4 q4 .. +3] and
//     element e feeds MFMA e of the four, so slot q4 of that MFMA is d = 16 i + 4 q4 + e; the
//     other operand is loaded with the same pairing.
//   accumulator fed back (P, dS): register v is the B operand of the MFMA whose slot q4 is row
//     4 q4 + v.  The matching A operand is X[4 q4 + v][64 j + 4 c16 .. +3]: element e feeds the
//     MFMA whose A row c16 is d = 64 j + 4 c16 + e, and C register w of accumulator (j, e) is
//     d = 64 j + 16 q4 + 4 w + e: a lane ends with 16 consecutive d per j and stores float4s.
// The sixteen-byte chunks of a row are permuted by chunk ^ (row & 7): the transposed read (16 chunks of a
// row) is free of bank conflicts, the row-major one (16 rows of a chunk column) takes two turns, half of the
// cycles in which LDS is active, which is a fifth of all.  Tiles have 32 rows, two LDS stages, filled by direct global -> LDS loads.
//
// N = 4096, H = 8, D = 128, G = 1024, forward + backward: plain fp32 fma kernels with a pre-pass
// for delta took 2890 us (10 TFLOP/s of the 14 D flops per pair), these 386 us (78; executed 100
// of the 154 TFLOP/s that a library fp32 product of 8192^3 reaches; forward 116 us and backward 272 with
// the matrix unit busy 69 and 79 % of the time a CU works).
// Problems of few rows: s2attn_f32_small.hip.
#include <cfloat>

#include "s2attn_bf16_common.h"
#include "s2attn_device.h"
#include "s2attn_f32_common.h"
#include "s2attn_launch.h"

namespace s2 {
namespace {

constexpr int kTile = 32;     // rows of a staged tile
constexpr int kWgRows = 64;   // rows a workgroup owns: 16 per wave

template <int D>
struct Lanes {
  static constexpr int kRow = D * 4;             // bytes of a tile row
  static constexpr int kTileBytes = kTile * kRow;
  int rm[2];   // row-major operand: byte offset for even / odd i, + 128 (i / 2)
  int tr[4];   // transposed operand of register v, + 256 j
  int st_row;  // staging: tile row of this lane's first 16 bytes, and its chunk
  int st_chunk;

  __device__ __forceinline__ void init(int lane, int w) {
    const int c16 = lane & 15, q4 = lane >> 4;
    rm[0] = c16 * kRow + ((q4 ^ (c16 & 7)) << 4);
    rm[1] = c16 * kRow + (((4 + q4) ^ (c16 & 7)) << 4);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 4 * q4 + v;
      tr[v] = row * kRow + ((c16 ^ (row & 7)) << 4);
    }
    constexpr int kChunks = D / 4;               // 16-byte chunks of a row: 16 or 32
    constexpr int kRowsPer = 64 / kChunks;       // rows one wave instruction fills: 4 or 2
    st_row = w * kRowsPer + lane / kChunks;
    st_chunk = (lane % kChunks) ^ (st_row & 7);
  }

  // X[16 RB + c16][16 i + 4 q4 ..]
  template <int RB>
  __device__ __forceinline__ f32x4 row(const char* tile, int i) const {
    return *reinterpret_cast<const f32x4*>(tile + rm[i & 1] + 16 * RB * kRow + 128 * (i >> 1));
  }
  // X[16 RB + 4 q4 + v][64 j + 4 c16 ..]
  template <int RB>
  __device__ __forceinline__ f32x4 col(const char* tile, int v, int j) const {
    return *reinterpret_cast<const f32x4*>(tile + tr[v] + 16 * RB * kRow + 256 * j);
  }

  // Stages rows i0 .. i0 + 31 of a run (clamped to its last row) of one head.
  __device__ __forceinline__ void stage(const KArgs& a, const Run& run, int s, const void* src, const TStride& st,
                                        int b, int head, int i0, uint32_t lds, int w) const {
    constexpr int kStep = 4 * (64 / (D / 4));    // rows the four waves fill together: 16 or 8
#pragma unroll
    for (int p = 0; p < kTile / kStep; ++p) {
      const int tok = run_token(a, run, i0 + p * kStep + st_row, s);
      dma16(static_cast<const char*>(src) + row_off(st, b, tok, head) * 4 + (st_chunk << 4), lds + (p * 4 + w) * 1024);
    }
  }
};

// acc[RB] += rows of the tile (16 RB + c16) against the wave's own 16 rows held in `own`.
template <int D>
__device__ __forceinline__ void scores(f32x4 (&acc)[2], const char* tile, const Lanes<D>& ln, const f32x4 (&own)[D / 16]) {
#pragma unroll
  for (int i = 0; i < D / 16; ++i) {
    const f32x4 x0 = ln.template row<0>(tile, i), x1 = ln.template row<1>(tile, i);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[0] = mfma4(x0[e], own[i][e], acc[0]);
      acc[1] = mfma4(x1[e], own[i][e], acc[1]);
    }
  }
}

// acc[j][e] += X^T W for the 32 rows of a tile: W = P or dS as it stands in the accumulators.
template <int D>
__device__ __forceinline__ void accumulate(f32x4 (&acc)[D / 64][4], const char* tile, const Lanes<D>& ln, const f32x4 (&wt)[2]) {
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int j = 0; j < D / 64; ++j) {
      const f32x4 x0 = ln.template col<0>(tile, v, j), x1 = ln.template col<1>(tile, v, j);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j][e] = mfma4(x0[e], wt[0][v], acc[j][e]);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j][e] = mfma4(x1[e], wt[1][v], acc[j][e]);
    }
}

// ---------------------------------------------------------------------------
// Forward.  A workgroup (4 waves) owns 64 query rows of one causal run, a wave 16 of them
// (queries on C columns, keys on registers): S^T = K Q^T, online softmax, O^T += V^T P^T.
// 64 rows and not 128: at D = 128 two such workgroups share a CU's LDS (64 KB each), and a
// layer of a few hundred tokens still spreads over the chip.
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(256, 2) fwd_f32_kernel(KArgs a, int T, Deal deal, int first_block) {
  using L = Lanes<D>;
  __shared__ __attribute__((aligned(1024))) char smem[4 * L::kTileBytes];   // [stage][K, V]
  fetch_args(a, deal);

  const int tid = thread_id(), lane = tid & 63, w = uni(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  int seq, rank;
  if (!decode_block(first_block + block_id(), T, deal, seq, rank)) return;
  const HeadPos at = head_of_seq(a, seq);
  const int s = uni(shift_of_head(a, at.h));
  Run run;
  int qt = T - 1 - rank;
  if (!run_of_tile(a, at.g, s, kWgRows, qt, run)) return;
  run.p0 = uni(run.p0); run.len = uni(run.len);
  const int i0 = uni(qt * kWgRows);
  const int qw0 = i0 + 16 * w, qrow = qw0 + c16;
  const int tok = run_token(a, run, qrow, s);
  const float c2 = a.scale_log2;

  L ln;
  ln.init(lane, w);
  const uint32_t base = lds_addr(smem);
  auto issue_tile = [&](int n) __attribute__((always_inline)) {
    const uint32_t dst = base + (n & 1) * 2 * L::kTileBytes;
    ln.stage(a, run, s, a.k, a.sk, at.b, at.c, n * kTile, dst, w);
    ln.stage(a, run, s, a.v, a.sv, at.b, at.c, n * kTile, dst + L::kTileBytes, w);
  };
  issue_tile(0);
  f32x4 qf[D / 16];
  load_own<D>(qf, a.q, row_off(a.sq, at.b, tok, at.h), q4);

  f32x4 o[D / 64][4];
#pragma unroll
  for (int j = 0; j < D / 64; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[j][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  // scaled (base 2) row maximum, and this lane's part of the row sum.  The maximum starts at the
  // lowest finite number: a row whose scores so far are all -inf then has weights of
  // exp2(-inf) = 0 and goes on with its later keys (from -inf they would be exp2(-inf + inf) = NaN)
  float m_run = -FLT_MAX, l_run = 0.f;

  const int n_tiles = uni((min(i0 + kWgRows, run.len) - 1) / kTile + 1);
  for (int n = 0; n < n_tiles; ++n) {
    wait_vmcnt0();
    __syncthreads();
    if (n + 1 < n_tiles) issue_tile(n + 1);
    const int j0 = n * kTile;
    if (j0 > qw0 + 15 || qw0 >= run.len) continue;   // wholly after this wave's queries, or no query at all
    const char* Ks = smem + (n & 1) * 2 * L::kTileBytes;
    const char* Vs = Ks + L::kTileBytes;
    f32x4 sc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    scores<D>(sc, Ks, ln, qf);
    const bool masked = j0 + kTile - 1 > qw0;
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float x = sc[kb][v] * c2;
        if (masked && j0 + 16 * kb + 4 * q4 + v > qrow) x = -INFINITY;
        sc[kb][v] = x;
        mx = fmaxf(mx, x);
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
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sc[kb][v] = exp2f(sc[kb][v] - m_run);
        l_run += sc[kb][v];
      }
    accumulate<D>(o, Vs, ln, sc);
  }

  const float l_tot = sum_cols(l_run);
  if (qrow >= run.len) return;
  store_row<D>(static_cast<float*>(a.o) + row_off(a.so, at.b, tok, at.h), o, 1.f / l_tot, q4);
  if (q4 == 0) a.lse[((size_t)at.b * a.H + at.h) * a.N + tok] = (m_run + log2f(l_tot)) * kLn2;
}

// ---------------------------------------------------------------------------
// Backward, one launch: the first n_kv blocks are dK/dV workgroups, the others dQ workgroups
// (independent of each other, and a small layer fills the chip with neither alone).
//   dK/dV: 64 keys of one kv head and part of its query heads (part_heads), a wave 16 keys on
//     the C columns with K and V in registers; walks the 32-row query tiles from the end of
//     the run to the diagonal, heads innermost.  S = Q K^T, dP - delta = dO V^T - delta,
//     dV^T += dO^T P, dK^T += Q^T dS.
//   dQ: 64 queries, a wave 16 of them; S^T = K Q^T, dP^T = V dO^T, dQ^T += K^T dS^T.
// delta_i = dO_i . O_i is formed here and not by a pre-pass: a dQ lane has its dO row in
// registers anyway, and a dK/dV workgroup forms the 32 sums of the next tile (8 threads a row)
// while the matrix unit works on the present one, which costs an O tile from L2 per query tile
// of 16 k MFMA cycles.  A launch saved is what counts at the small sizes.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void bwd_dkdv_block(const KArgs& a, char* smem, float* rows_s, int block, int T, const Deal& deal) {
  using L = Lanes<D>;
  const int tid = thread_id(), lane = tid & 63, w = uni(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  int seq, kt;
  if (!decode_block(block, T, deal, seq, kt)) return;   // key tile 0 is the heaviest
  const KvPos at = kv_of_seq(a, seq);
  int h_lo, nheads, s;
  part_heads(a, at.c, at.part, h_lo, nheads, s);
  Run run;
  if (!run_of_tile(a, at.g, s, kWgRows, kt, run)) return;
  run.p0 = uni(run.p0); run.len = uni(run.len);
  const int j0 = uni(kt * kWgRows);
  const int kw0 = j0 + 16 * w, key = kw0 + c16;
  const int tok = run_token(a, run, key, s);
  const int it_first = j0 / kTile, it_last = uni((run.len - 1) / kTile);
  const int n_iter = nheads * (it_last - it_first + 1);
  const float c2 = a.scale_log2;

  L ln;
  ln.init(lane, w);
  const uint32_t base = lds_addr(smem);
  auto issue_tile = [&](int hh, int it, int stage) __attribute__((always_inline)) {
    const uint32_t dst = base + stage * 2 * L::kTileBytes;
    ln.stage(a, run, s, a.q, a.sq, at.b, h_lo + hh, it * kTile, dst, w);
    ln.stage(a, run, s, a.dout, a.so, at.b, h_lo + hh, it * kTile, dst + L::kTileBytes, w);
  };
  // row terms of a tile: thread -> (row tid / 8, every eighth float4 of it)
  f32x4 ov[D / 32], gv[D / 32];
  float lse = 0.f;
  auto load_rows = [&](int hh, int it) __attribute__((always_inline)) {
    const int t = run_token(a, run, it * kTile + (tid >> 3), s);
    const size_t off = row_off(a.so, at.b, t, h_lo + hh) + 4 * (tid & 7);
#pragma unroll
    for (int k = 0; k < D / 32; ++k) {
      ov[k] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.o) + off + 32 * k);
      gv[k] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.dout) + off + 32 * k);
    }
    lse = a.lse[((size_t)at.b * a.H + h_lo + hh) * a.N + t];
  };
  auto finish_rows = [&](int stage) __attribute__((always_inline)) {
    float x = 0.f;
#pragma unroll
    for (int k = 0; k < D / 32; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) x = fmaf(ov[k][e], gv[k][e], x);
    x += __shfl_xor(x, 1);
    x += __shfl_xor(x, 2);
    x += __shfl_xor(x, 4);
    if ((tid & 7) == 0) {
      rows_s[stage * 2 * kTile + (tid >> 3)] = lse * kLog2e;
      rows_s[stage * 2 * kTile + kTile + (tid >> 3)] = x;
    }
  };

  f32x4 kf[D / 16], vf[D / 16], dk[D / 64][4], dv[D / 64][4];
  load_own<D>(kf, a.k, row_off(a.sk, at.b, tok, at.c), q4);
  load_own<D>(vf, a.v, row_off(a.sv, at.b, tok, at.c), q4);
#pragma unroll
  for (int j = 0; j < D / 64; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) { dk[j][e] = f32x4{0.f, 0.f, 0.f, 0.f}; dv[j][e] = dk[j][e]; }

  int hh = 0, it = it_last;
  if (n_iter > 0) {
    issue_tile(0, it_last, 0);
    load_rows(0, it_last);
    finish_rows(0);
  }
  for (int n = 0; n < n_iter; ++n) {
    const int stage = n & 1;
    const int q0 = it * kTile;
    if (++hh == nheads) { hh = 0; --it; }    // the next tile
    wait_vmcnt0();
    __syncthreads();
    if (n + 1 < n_iter) {
      issue_tile(hh, it, stage ^ 1);
      load_rows(hh, it);
    }
    if (q0 + kTile - 1 >= kw0 && kw0 < run.len) {   // else: all queries of the tile before this wave's keys, or no key
      const char* Qs = smem + stage * 2 * L::kTileBytes;
      const char* dOs = Qs + L::kTileBytes;
      const float* lse2 = rows_s + stage * 2 * kTile + 4 * q4;
      f32x4 sc[2], dp[2];
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        sc[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
        dp[qb] = -*reinterpret_cast<const f32x4*>(lse2 + kTile + 16 * qb);
      }
      scores<D>(sc, Qs, ln, kf);
      scores<D>(dp, dOs, ln, vf);
      const bool masked = kw0 + 15 > q0 || q0 + kTile > run.len;
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(lse2 + 16 * qb);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = q0 + 16 * qb + 4 * q4 + v;
          float p = exp2f(fmaf(sc[qb][v], c2, -l4[v]));
          if (masked && (key > i || i >= run.len)) p = 0.f;
          sc[qb][v] = p;
          dp[qb][v] *= p;
        }
      }
      accumulate<D>(dv, dOs, ln, sc);
      accumulate<D>(dk, Qs, ln, dp);
    }
    if (n + 1 < n_iter) finish_rows(stage ^ 1);
  }

  if (key >= run.len) return;
  if (a.dkv_partial) {   // contiguous fp32 partial of this part, summed by the combine pass
    const size_t elems = (size_t)a.B * a.N * a.Hkv * D;
    float* dst = a.dkv_partial + at.part * elems + ((size_t)((size_t)at.b * a.N + tok) * a.Hkv + at.c) * D;
    store_row<D>(dst, dk, a.scale, q4);
    store_row<D>(dst + a.parts * elems, dv, 1.f, q4);
  } else {
    store_row<D>(static_cast<float*>(a.dk) + row_off(a.sdk, at.b, tok, at.c), dk, a.scale, q4);
    store_row<D>(static_cast<float*>(a.dv) + row_off(a.sdv, at.b, tok, at.c), dv, 1.f, q4);
  }
}

template <int D>
__device__ __forceinline__ void bwd_dq_block(const KArgs& a, char* smem, int block, int T, const Deal& deal) {
  using L = Lanes<D>;
  const int tid = thread_id(), lane = tid & 63, w = uni(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  int seq, rank;
  if (!decode_block(block, T, deal, seq, rank)) return;
  const HeadPos at = head_of_seq(a, seq);
  const int s = uni(shift_of_head(a, at.h));
  Run run;
  int qt = T - 1 - rank;
  if (!run_of_tile(a, at.g, s, kWgRows, qt, run)) return;
  run.p0 = uni(run.p0); run.len = uni(run.len);
  const int i0 = uni(qt * kWgRows);
  const int qw0 = i0 + 16 * w, qrow = qw0 + c16;
  const int tok = run_token(a, run, qrow, s);
  const float c2 = a.scale_log2;

  L ln;
  ln.init(lane, w);
  const uint32_t base = lds_addr(smem);
  auto issue_tile = [&](int n) __attribute__((always_inline)) {
    const uint32_t dst = base + (n & 1) * 2 * L::kTileBytes;
    ln.stage(a, run, s, a.k, a.sk, at.b, at.c, n * kTile, dst, w);
    ln.stage(a, run, s, a.v, a.sv, at.b, at.c, n * kTile, dst + L::kTileBytes, w);
  };
  issue_tile(0);
  f32x4 qf[D / 16], gf[D / 16], dq[D / 64][4];
  float delta = 0.f;
  {
    f32x4 of[D / 16];
    load_own<D>(qf, a.q, row_off(a.sq, at.b, tok, at.h), q4);
    load_own<D>(gf, a.dout, row_off(a.so, at.b, tok, at.h), q4);
    load_own<D>(of, a.o, row_off(a.so, at.b, tok, at.h), q4);
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) delta = fmaf(of[i][e], gf[i][e], delta);
    delta = sum_cols(delta);
  }
  const float lse2 = a.lse[((size_t)at.b * a.H + at.h) * a.N + tok] * kLog2e;
#pragma unroll
  for (int j = 0; j < D / 64; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) dq[j][e] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int n_tiles = uni((min(i0 + kWgRows, run.len) - 1) / kTile + 1);
  for (int n = 0; n < n_tiles; ++n) {
    wait_vmcnt0();
    __syncthreads();
    if (n + 1 < n_tiles) issue_tile(n + 1);
    const int j0 = n * kTile;
    if (j0 > qw0 + 15 || qw0 >= run.len) continue;
    const char* Ks = smem + (n & 1) * 2 * L::kTileBytes;
    const char* Vs = Ks + L::kTileBytes;
    f32x4 sc[2], dp[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      sc[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
      dp[kb] = f32x4{-delta, -delta, -delta, -delta};
    }
    scores<D>(sc, Ks, ln, qf);
    scores<D>(dp, Vs, ln, gf);
    const bool masked = j0 + kTile - 1 > qw0;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float p = exp2f(fmaf(sc[kb][v], c2, -lse2));
        if (masked && j0 + 16 * kb + 4 * q4 + v > qrow) p = 0.f;
        dp[kb][v] *= p;
      }
    accumulate<D>(dq, Ks, ln, dp);
  }
  if (qrow >= run.len) return;
  store_row<D>(static_cast<float*>(a.dq) + row_off(a.sdq, at.b, tok, at.h), dq, a.scale, q4);
}

template <int D>
__global__ void __launch_bounds__(256, 2)
bwd_f32_kernel(KArgs a, int n_kv, int T, Deal deal_kv, Deal deal_q, int first_block) {
  __shared__ __attribute__((aligned(1024))) char smem[4 * Lanes<D>::kTileBytes];   // [stage][Q, dO] or [stage][K, V]
  __shared__ __attribute__((aligned(16))) float rows_s[2 * 2 * kTile];             // [stage][lse * log2(e), delta]
  const int block = first_block + block_id();
  if (block < n_kv)
    bwd_dkdv_block<D>(a, smem, rows_s, block, T, deal_kv);
  else
    bwd_dq_block<D>(a, smem, block - n_kv, T, deal_q);
}

template <int D>
int launch_fwd_t(const KArgs& a, hipStream_t st) {
  const int T = ragged_tiles(a, kWgRows);
  const Grid g = grid_of(T, a.B * a.H * a.NG, a.r, 64);
  return launch_blocks(fwd_f32_kernel<D>, g.blocks, 256, st, a, T, g.deal);
}

template <int D>
int launch_bwd_t(const KArgs& a, bool dq_last, hipStream_t st) {
  const int T = ragged_tiles(a, kWgRows);
  const Grid kv = grid_of(T, a.B * a.Hkv * a.NG * a.parts, 1, 64), q = grid_of(T, a.B * a.H * a.NG, a.r, 64);
  const int n_first = dq_last ? kv.blocks : kv.blocks + q.blocks;
  const int rc = launch_blocks(bwd_f32_kernel<D>, n_first, 256, st, a, kv.blocks, T, kv.deal, q.deal);
  if (rc != 0 || !dq_last) return rc;
  return launch_blocks(bwd_f32_kernel<D>, q.blocks, 256, st, a, 0, T, kv.deal, q.deal);
}

// Few workgroups of 64 rows: 16 rows to a workgroup and its waves on different tiles (s2attn_f32_small.hip).
// Times: us here and there.
// Forward up to one workgroup per CU (H = 4, D = 128, groups of 500, N = 1000: 44.7 and 16.7; H = 8,
// N = 2048, groups of 512, 256 workgroups: 46.0 and 38.4; groups of 256, 512 workgroups: 34.9 and 42.5), in
// groups of one workgroup or less up to a quarter of that (groups of 64, H = 4, D = 64, N = 256, 16 workgroups:
// 6.4 and 4.7; N = 2560, 160 workgroups: 6.8 and 7.2).  In groups of two workgroups, whose chains are short, the busiest
// XCD's share of the workgroups of 16 rows counts (three to a CU, D = 64 four; groups of 128, D = 128: 11 sequences, 88
// workgroups, 14.9 and 13.2; 16, 128 workgroups, 15.2 and 17.5; D = 64 10.1 and 10.0).  And not for long runs, which the
// tiles in LDS serve better than the caches (H = 2, one group, D = 128: N = 4500 491 and 456, 5500 626 and 676; D = 64,
// H = 1: 10000 1046 and 1033, 16000 2366 and 2611).
bool small_fwd(const KArgs& a) {
  const int n_seq = a.B * a.H * a.NG;
  const long long n = (long long)n_seq * ragged_tiles(a, kWgRows);
  if (n > (a.G > kWgRows ? 256 : 64) || (long long)a.G * a.D > 4608 * 128) return false;
  return a.G > 2 * kWgRows || most_of_an_xcd(n_seq) * ((a.G + 15) / 16) <= (a.D == 64 ? 128 : 100);
}
// Backward, which reads every tile in four or five forms there, from the caches: up to half a workgroup per CU
// in groups of more than 256, groups of a few tiles an eighth (of 250 to 256 three eighths) unless several query heads
// to a kv head make dK/dV's chains long again.  H = 4, D = 64, groups of 256, N = 1024 (64 workgroups): 26.2 and 19.7;
// D = 128, groups of 512, N = 2048 (128) 82.2 and 72.1, N = 2560 (160) 113 and 134; groups of 64, N = 256 (16) 14.6 and
// 10.6, N = 1024 (64) 15.8 and 17.9; groups of 250, 24 sequences (96) 43.8 and 36.8, 32 (128) 44.1 and 46.8; H = 8,
// Hkv = 2, groups of 128, N = 1024 (128) 47.7 and 38.8.
// Long chains up to one workgroup per CU of the busiest XCD (D = 128; groups of 1000: eight sequences 159 and 117, sixteen
// 235 and 214, twenty 223 and 312; of 1250: eight 238 and 174, ten 265 and 326; of 1500: eight 312 and 229, twelve 326
// and 446; 2048: one to eight 470 and 400; 2500: 509 and 585; 4096: 1014 and 1490; 8192: 3860 and 5780).
bool small_bwd(const KArgs& a) {
  const int n_seq = a.B * a.H * a.NG, T = ragged_tiles(a, kWgRows);
  if (a.G >= 1000) return (long long)most_of_an_xcd(n_seq) * T <= 32;
  return (long long)n_seq * T <= (a.G > 256 || a.r >= 4 ? 128 : a.G >= 250 ? 96 : 32);
}

}  // namespace

int launch_fwd_f32(const KArgs& a, hipStream_t st) {
  if (small_fwd(a)) return launch_fwd_f32_small(a, st);
  return a.D == 64 ? launch_fwd_t<64>(a, st) : launch_fwd_t<128>(a, st);
}

int launch_bwd_f32(const KArgs& a, bool dq_last, hipStream_t st) {
  if (small_bwd(a)) return launch_bwd_f32_small(a, dq_last, st);
  return a.D == 64 ? launch_bwd_t<64>(a, dq_last, st) : launch_bwd_t<128>(a, dq_last, st);
}

}  // namespace s2
