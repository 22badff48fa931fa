// bf16 S2-Attn kernels (forward; backward) for problems of few rows (D = 128).
//
// What bounds a small problem is the chain of tiles of one workgroup, and the launches, while most of the
// chip is idle.  Here a workgroup owns 32 rows and its four waves share out the tiles of 32 rows that
// these meet: four times the workgroups of the other kernels (128 rows) and a quarter of their chain.  Every
// wave stages its own tiles into its own part of LDS (the next tile while it works on one, no barrier); the
// waves' sums meet in LDS once, at the end.  The backward forms delta itself (a dQ lane has its dO rows in registers; a
// dK/dV wave forms that of each query tile it takes) and so is one launch and not two.
//
// v_mfma_f32_16x16x32_bf16, lane l: c16 = l % 16, q4 = l / 16 (operand layout: s2attn_bf16_common.h).
//   forward, dQ:  S^T = K Q^T, dP^T = V dO^T (keys on registers, queries on lanes), O^T += V^T P^T, dQ^T += K^T dS^T
//   dK/dV:        S = Q K^T, dP = dO V^T (queries on registers, keys on lanes), dV^T += dO^T P, dK^T += Q^T dS
// Any even group size, any shift; tiles that are not 32 consecutive tokens are staged row by row.
#include "s2attn_bf16_common.h"
#include "s2attn_device.h"
#include "s2attn_launch.h"

namespace s2 {
namespace {

constexpr int kRows = 32;                            // rows of a workgroup, and of a tile
constexpr int kWaves = 4;
constexpr int kTileBytes = kRows * kRowBytes;        // 8 KB
constexpr int kRingBytes = 2 * 2 * kTileBytes;       // two stages of two tensors
constexpr int kBlockFloats = kRows * (128 + 4);      // a wave's 32 x 128 sums; rows four floats apart in the banks
constexpr int kSmemFwd = kWaves * kRingBytes;
constexpr int kSmemBwd = 2 * kWaves * kBlockFloats * 4;
static_assert(kSmemFwd >= kWaves * kBlockFloats * 4 && kSmemBwd >= kSmemFwd, "rings and sums share the memory");

// A wave's staging of tiles of two tensors x and y with the same rows: eight pairs of loads, four rows each.
struct Ring {
  uint64_t xb, yb;                                   // head bases
  long long x_row, y_row;                            // bytes of a token step
  uint32_t lds;                                      // this wave's ring
  int sub, chunk;                                    // this lane's row of the four, its 16 bytes of the row in LDS
  uint32_t x_lane[4], y_lane[4];                     // lane offset of pair p (by p % 4) of a tile of consecutive tokens
  // the tile being issued
  bool pending;
  uint64_t x0, y0;
  uint32_t dst;

  __device__ __forceinline__ void init(const TStride& sx, const TStride& sy, uint32_t base, int lane) {
    x_row = sx.t * 2; y_row = sy.t * 2;
    lds = base;
    sub = lane >> 4;
    chunk = (lane & 15) ^ (sub << 2);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint32_t c = (uint32_t)(chunk ^ p) << 4;   // chunk ^ swz(4 p + sub)
      x_lane[p] = (uint32_t)sub * (uint32_t)x_row + c;
      y_lane[p] = (uint32_t)sub * (uint32_t)y_row + c;
    }
  }
  __device__ __forceinline__ void head(const void* x, const TStride& sx, int hx, const void* y, const TStride& sy, int hy, int b) {
    xb = uni64(reinterpret_cast<uint64_t>(x) + row_off(sx, b, 0, hx) * 2);
    yb = uni64(reinterpret_cast<uint64_t>(y) + row_off(sy, b, 0, hy) * 2);
  }
  // Rows i0 .. i0 + 31 of the run into stage `stage`, where `want`: consecutive tokens by the pair() calls that
  // follow, others at once, row by row (rows past the end repeat the last row).
  __device__ __forceinline__ void begin(const KArgs& a, const Run& run, int s, int i0, int stage, bool want) {
    dst = lds + stage * 2 * kTileBytes;
    pending = want;
    if (!want) return;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // every read of the stage is done
    const uint32_t tok0 = (uint32_t)uni(token_of(run.p0 + i0, s, a.N));
    x0 = xb + tok0 * x_row;
    y0 = yb + tok0 * y_row;
    if (i0 + kRows > run.len || (int)tok0 + kRows > a.N) {
      pending = false;
#pragma unroll 1
      for (int p = 0; p < 8; ++p) {
        const int tok = run_token(a, run, i0 + 4 * p + sub, s);
        const uint32_t c = (uint32_t)(chunk ^ (p & 3)) << 4;
        dma16(reinterpret_cast<const char*>(xb) + tok * x_row + c, dst + 1024 * p);
        dma16(reinterpret_cast<const char*>(yb) + tok * y_row + c, dst + 1024 * p + kTileBytes);
      }
    }
  }
  __device__ __forceinline__ void pair(int p) const {
    if (pending) {
      dma16s(x0 + 4 * p * x_row, x_lane[p & 3], dst + 1024 * p);
      dma16s(y0 + 4 * p * y_row, y_lane[p & 3], dst + 1024 * p + kTileBytes);
    }
  }
  __device__ __forceinline__ void all_pairs() const {
#pragma unroll
    for (int p = 0; p < 8; ++p) pair(p);
  }
};

// The tile in flight has landed.
__device__ __forceinline__ void wait_tile() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A wave's own 32 rows as B operands: X[row c16 + 16 b][32 k + 8 q4 ..].
__device__ __forceinline__ void load_own(bf16x8 (&f)[4][2], const KArgs& a, const void* src, const TStride& st, const Run& run, int s,
                                         int b, int head, int i0, int lane) {
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    const int tok = run_token(a, run, i0 + 16 * rb + (lane & 15), s);
    const bf16x8* p = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(src) + row_off(st, b, tok, head));
#pragma unroll
    for (int k = 0; k < 4; ++k) f[k][rb] = p[4 * k + (lane >> 4)];
  }
}

// Waits for loads here: a first use inside the loop would have the compiler wait there for all younger
// loads too, in every pass.
__device__ __forceinline__ void arrived(bf16x8 (&f)[4][2]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(f[k][0]), "+v"(f[k][1]));
}

// acc[rb][cb] += X Y^T: 16-row blocks rb of the tile X against the wave's own rows 16 cb ..
// (each(k) after the MFMAs of step k: the loads of the next tile go out between the steps, for the four waves of
// a CU together wait for its 64 bytes a clock otherwise)
template <class Each>
__device__ __forceinline__ void products(f32x4 (&acc)[2][2], const char* X, const LaneOffsets16& lo, const bf16x8 (&own)[4][2], Each each) {
  bf16x8 f[4][2];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    f[k][0] = frag_rm<0>(X, lo, k);
    f[k][1] = frag_rm<16>(X, lo, k);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) acc[rb][cb] = mfma16(f[k][rb], own[k][cb], acc[rb][cb]);
    each(k);
  }
}

// acc^T (128 x 32) += X^T W for the 32 rows of the tile X, W as B operands of 16 columns
__device__ __forceinline__ void accumulate(f32x4 (&acc)[8][2], const char* X, const LaneOffsets16& lo, const bf16x8 (&w)[2]) {
#pragma unroll
  for (int db = 0; db < 8; ++db) {
    const bf16x8 f = frag_tr<0>(X, lo, db);
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) acc[db][cb] = mfma16(f, w[cb], acc[db][cb]);
  }
}

__device__ __forceinline__ void zero(f32x4 (&acc)[8][2]) {
#pragma unroll
  for (int db = 0; db < 8; ++db) acc[db][0] = acc[db][1] = zero4();
}

__device__ __forceinline__ void put_block(float* block, const f32x4 (&acc)[8][2], int lane) {
#pragma unroll
  for (int db = 0; db < 8; ++db)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
      *reinterpret_cast<f32x4*>(block + (16 * cb + (lane & 15)) * 132 + 16 * db + 4 * (lane >> 4)) = acc[db][cb];
}

// Columns 8 c .. +7 of row `row` of the sum of the waves' blocks, each times its factor.
__device__ __forceinline__ void sum_blocks(f32x4 (&x)[2], const float* blocks, int row, int c, const float (&factor)[kWaves]) {
  x[0] = x[1] = zero4();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const f32x4* p = reinterpret_cast<const f32x4*>(blocks + w * kBlockFloats + row * 132 + 8 * c);
    x[0] += p[0] * factor[w];
    x[1] += p[1] * factor[w];
  }
}

// delta of 16 rows, dO . O: the diagonal of the product of the two, which lane (q4, c16 = 4 q4 + v) holds in
// register v.  Four matrix instructions take the place of 32 conversions and products per lane and row block.
__device__ __forceinline__ f32x4 row_dots(const bf16x8 (&x)[4][2], const bf16x8 (&y)[4][2], int rb) {
  f32x4 d = zero4();
#pragma unroll
  for (int k = 0; k < 4; ++k) d = mfma16(x[k][rb], y[k][rb], d);
  return d;
}
// by register: delta of row 4 q4 + v in register v of every lane
__device__ __forceinline__ f32x4 diag_rows(f32x4 d, int lane) {
  const int at = 20 * (lane >> 4);
  f32x4 r;
#pragma unroll
  for (int v = 0; v < 4; ++v) r[v] = __shfl(d[v], at + v);
  return r;
}
// by lane: delta of row c16 in every lane of that column
__device__ __forceinline__ float diag_cols(f32x4 d, int lane) {
  const int c16 = lane & 15, v = c16 & 3;
  const float x = v == 0 ? d[0] : v == 1 ? d[1] : v == 2 ? d[2] : d[3];
  return __shfl(x, 16 * (c16 >> 2) + c16);
}

__global__ void __launch_bounds__(64 * kWaves, 1) fwd_small_kernel(KArgs a, int T, Deal deal, int first_block) {
  __shared__ __attribute__((aligned(1024))) char smem[kSmemFwd];
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
  qt = uni(qt); run.p0 = uni(run.p0); run.len = uni(run.len);
  const int i0 = qt * kRows, qrow = i0 + c16;
  const float c2 = a.scale_log2;

  Ring ring;
  ring.init(a.sk, a.sv, lds_addr(smem) + w * kRingBytes, lane);
  ring.head(a.k, a.sk, at.c, a.v, a.sv, at.c, at.b);
  const char* base = smem + w * kRingBytes;
  bf16x8 qf[4][2];
  load_own(qf, a, a.q, a.sq, run, s, at.b, at.h, i0, lane);
  ring.begin(a, run, s, w * kRows, 0, w <= qt);
  ring.all_pairs();

  LaneOffsets16 lo;
  init_lane_offsets(lo, lane);
  f32x4 o[8][2];
  zero(o);
  // scaled (base 2) maximum and this lane's part of the row sum; finite from the start, so that a row
  // whose scores so far are all -inf has weights of zero
  float m_run[2] = {-3.402823466e38f, -3.402823466e38f}, l_run[2] = {0.f, 0.f};
  arrived(qf);
  int stage = 0;
  for (int jt = w; jt <= qt; jt += kWaves, stage ^= 1) {
    wait_tile();
    ring.begin(a, run, s, (jt + kWaves) * kRows, stage ^ 1, jt + kWaves <= qt);
    const char* Ks = base + stage * 2 * kTileBytes;
    const char* Vs = Ks + kTileBytes;
    f32x4 sc[2][2] = {{zero4(), zero4()}, {zero4(), zero4()}};
    products(sc, Ks, lo, qf, [&](int k) { ring.pair(2 * k); ring.pair(2 * k + 1); });
    bf16x8 pf[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float x = sc[kb][qb][e] * c2;
          if (jt == qt && 16 * kb + 4 * q4 + e > c16 + 16 * qb) x = -INFINITY;
          sc[kb][qb][e] = x;
          mx = fmaxf(mx, x);
        }
      mx = max_of_4(mx);
      if (__builtin_amdgcn_ballot_w64(mx > m_run[qb]) != 0) {
        const float m_new = fmaxf(m_run[qb], mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
        m_run[qb] = m_new;
        l_run[qb] *= alpha;
#pragma unroll
        for (int db = 0; db < 8; ++db) o[db][qb] *= alpha;
      }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sc[kb][qb][e] = __builtin_amdgcn_exp2f(sc[kb][qb][e] - m_run[qb]);
          l_run[qb] += sc[kb][qb][e];
        }
      pf[qb] = pack8(sc[0][qb], sc[1][qb]);
    }
    accumulate(o, Vs, lo, pf);
  }
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) l_run[qb] = sum_of_4(l_run[qb]);
  __syncthreads();   // the rings are done with
  float* blocks = reinterpret_cast<float*>(smem);
  put_block(blocks + w * kBlockFloats, o, lane);
  if (q4 == 0)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      max_s[w][16 * qb + c16] = m_run[qb];
      sum_s[w][16 * qb + c16] = l_run[qb];
    }
  __syncthreads();

#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int row = 16 * pass + (tid >> 4), c = tid & 15;
    if (i0 + row >= run.len) break;
    float m = max_s[0][row], factor[kWaves], l = 0.f;
#pragma unroll
    for (int x = 1; x < kWaves; ++x) m = fmaxf(m, max_s[x][row]);
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      factor[x] = __builtin_amdgcn_exp2f(max_s[x][row] - m);
      l = fmaf(sum_s[x][row], factor[x], l);
    }
    f32x4 r[2];
    sum_blocks(r, blocks, row, c, factor);
    const float inv = 1.f / l;
    const int t = token_of(run.p0 + i0 + row, s, a.N);
    *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(a.o) + row_off(a.so, at.b, t, at.h) + 8 * c) = pack8(r[0] * inv, r[1] * inv);
    if (c == 0) a.lse[((size_t)at.b * a.H + at.h) * a.N + t] = (m + __builtin_amdgcn_logf(l)) * kLn2;
  }
}

// dK/dV of 32 keys; the waves share out the query tiles of all query heads of the part.
__device__ __forceinline__ void dkdv_small_block(const KArgs& a, char* smem, int block, int T, const Deal& deal) {
  const int tid = thread_id(), lane = tid & 63, w = uni(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  int seq, kt;
  if (!decode_block(block, T, deal, seq, kt)) return;
  const KvPos at = kv_of_seq(a, seq);
  int h_lo, nheads, s;
  part_heads(a, at.c, at.part, h_lo, nheads, s);
  Run run;
  if (!run_of_tile(a, at.g, s, kRows, kt, run)) return;
  kt = uni(kt); run.p0 = uni(run.p0); run.len = uni(run.len);
  const int j0 = kt * kRows, key = j0 + c16;
  const int nq = uni((run.len - 1) / kRows) - kt + 1;   // query tiles of a head, from the diagonal on
  const float c2 = a.scale_log2;

  Ring ring;
  ring.init(a.sq, a.so, lds_addr(smem) + w * kRingBytes, lane);
  const char* base = smem + w * kRingBytes;
  bf16x8 of[4][2];
  float lse[2];
  // O and lse of tile `it` from the diagonal of head h_lo + hh
  auto load_rows = [&](int hh, int it) __attribute__((always_inline)) {
    const int h = h_lo + hh, q0 = j0 + it * kRows;
    load_own(of, a, a.o, a.so, run, s, at.b, h, q0, lane);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
      lse[rb] = a.lse[((size_t)at.b * a.H + h) * a.N + run_token(a, run, q0 + 16 * rb + c16, s)];
  };
  auto settle = [&](int& hh, int& it) __attribute__((always_inline)) {
    while (hh < nheads && it >= nq) { it -= nq; ++hh; }
  };
  bf16x8 kf[4][2], vf[4][2];
  load_own(kf, a, a.k, a.sk, run, s, at.b, at.c, j0, lane);
  load_own(vf, a, a.v, a.sv, run, s, at.b, at.c, j0, lane);
  LaneOffsets16 lo;
  init_lane_offsets(lo, lane);
  f32x4 dk[8][2], dv[8][2];
  zero(dk);
  zero(dv);
  arrived(kf);
  arrived(vf);
  // the wave's tiles (head hn, query tile in), every fourth; a pass issues one and works on the one before
  int hn = 0, in = w, q0 = 0, stage = 0;
  bool cur = false, diagonal = false;
  settle(hn, in);
  while (true) {
    const bool more = hn < nheads;
    const char* Qs = base + stage * 2 * kTileBytes;
    const char* dOs = Qs + kTileBytes;
    if (cur) {
      wait_tile();
      arrived(of);
      asm volatile("" : "+v"(lse[0]), "+v"(lse[1]));
    }
    if (more) ring.head(a.q, a.sq, h_lo + hn, a.dout, a.so, h_lo + hn, at.b);
    ring.begin(a, run, s, j0 + in * kRows, stage ^ 1, more);
    if (!cur) ring.all_pairs();
    bf16x8 gf[4][2];
    f32x4 delta[2], lse2[2];
    if (cur) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        gf[k][0] = frag_rm<0>(dOs, lo, k);
        gf[k][1] = frag_rm<16>(dOs, lo, k);
      }
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        delta[rb] = diag_rows(row_dots(of, gf, rb), lane);
        const float l = lse[rb] * kLog2e;
#pragma unroll
        for (int e = 0; e < 4; ++e) lse2[rb][e] = __shfl(l, 4 * q4 + e);
      }
    }
    if (more) load_rows(hn, in);
    if (cur) {
      f32x4 sc[2][2] = {{zero4(), zero4()}, {zero4(), zero4()}}, dp[2][2];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) dp[rb][0] = dp[rb][1] = -delta[rb];
      products(sc, Qs, lo, kf, [&](int k) { ring.pair(k); });
#pragma unroll
      for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int cb = 0; cb < 2; ++cb) dp[rb][cb] = mfma16(gf[k][rb], vf[k][cb], dp[rb][cb]);
        ring.pair(4 + k);
      }
      const bool masked = diagonal || q0 + kRows > run.len;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = q0 + 16 * rb + 4 * q4 + e;
#pragma unroll
          for (int cb = 0; cb < 2; ++cb) {
            float p = __builtin_amdgcn_exp2f(fmaf(sc[rb][cb][e], c2, -lse2[rb][e]));
            if (masked && (key + 16 * cb > row || row >= run.len)) p = 0.f;
            sc[rb][cb][e] = p;
            dp[rb][cb][e] *= p;
          }
        }
      const bf16x8 pf[2] = {pack8(sc[0][0], sc[1][0]), pack8(sc[0][1], sc[1][1])};
      const bf16x8 ds[2] = {pack8(dp[0][0], dp[1][0]), pack8(dp[0][1], dp[1][1])};
      accumulate(dv, dOs, lo, pf);
      accumulate(dk, Qs, lo, ds);
    }
    if (!more) break;
    cur = true;
    diagonal = in == 0;
    q0 = j0 + in * kRows;
    stage ^= 1;
    in += kWaves;
    settle(hn, in);
  }
  __syncthreads();   // the rings are done with
  float* blocks = reinterpret_cast<float*>(smem);
  float* dv_blocks = blocks + kWaves * kBlockFloats;
  put_block(blocks + w * kBlockFloats, dk, lane);
  put_block(dv_blocks + w * kBlockFloats, dv, lane);
  __syncthreads();
  const float scale[kWaves] = {a.scale, a.scale, a.scale, a.scale}, one[kWaves] = {1.f, 1.f, 1.f, 1.f};
  const size_t elems = (size_t)a.B * a.N * a.Hkv * 128;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int row = 16 * pass + (tid >> 4), c = tid & 15;
    if (j0 + row >= run.len) break;
    const int t = token_of(run.p0 + j0 + row, s, a.N);
    f32x4 x[2], y[2];
    sum_blocks(x, blocks, row, c, scale);
    sum_blocks(y, dv_blocks, row, c, one);
    if (a.dkv_partial) {   // contiguous fp32 partial of this part, summed by the combine pass
      f32x4* dst = reinterpret_cast<f32x4*>(a.dkv_partial + at.part * elems + ((size_t)((size_t)at.b * a.N + t) * a.Hkv + at.c) * 128 + 8 * c);
      dst[0] = x[0];
      dst[1] = x[1];
      dst += a.parts * elems / 4;
      dst[0] = y[0];
      dst[1] = y[1];
    } else {
      *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(a.dk) + row_off(a.sdk, at.b, t, at.c) + 8 * c) = pack8(x[0], x[1]);
      *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(a.dv) + row_off(a.sdv, at.b, t, at.c) + 8 * c) = pack8(y[0], y[1]);
    }
  }
}

// dQ of 32 query rows; the waves share out the key tiles.
__device__ __forceinline__ void dq_small_block(const KArgs& a, char* smem, int block, int T, const Deal& deal) {
  const int tid = thread_id(), lane = tid & 63, w = uni(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  int seq, rank;
  if (!decode_block(block, T, deal, seq, rank)) return;
  const HeadPos at = head_of_seq(a, seq);
  const int s = uni(shift_of_head(a, at.h));
  Run run;
  int qt = T - 1 - rank;
  if (!run_of_tile(a, at.g, s, kRows, qt, run)) return;
  qt = uni(qt); run.p0 = uni(run.p0); run.len = uni(run.len);
  const int i0 = qt * kRows;
  const float c2 = a.scale_log2;

  Ring ring;
  ring.init(a.sk, a.sv, lds_addr(smem) + w * kRingBytes, lane);
  ring.head(a.k, a.sk, at.c, a.v, a.sv, at.c, at.b);
  const char* base = smem + w * kRingBytes;
  bf16x8 qf[4][2], gf[4][2];
  float delta[2], lse2[2];
  {
    bf16x8 of[4][2];
    load_own(gf, a, a.dout, a.so, run, s, at.b, at.h, i0, lane);
    load_own(of, a, a.o, a.so, run, s, at.b, at.h, i0, lane);
    load_own(qf, a, a.q, a.sq, run, s, at.b, at.h, i0, lane);
    ring.begin(a, run, s, w * kRows, 0, w <= qt);
    ring.all_pairs();
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      delta[qb] = diag_cols(row_dots(of, gf, qb), lane);
      lse2[qb] = a.lse[((size_t)at.b * a.H + at.h) * a.N + run_token(a, run, i0 + 16 * qb + c16, s)] * kLog2e;
    }
  }
  asm volatile("" : "+v"(delta[0]), "+v"(delta[1]), "+v"(lse2[0]), "+v"(lse2[1]));
  arrived(qf);
  arrived(gf);
  LaneOffsets16 lo;
  init_lane_offsets(lo, lane);
  f32x4 dq[8][2];
  zero(dq);
  int stage = 0;
  for (int jt = w; jt <= qt; jt += kWaves, stage ^= 1) {
    wait_tile();
    ring.begin(a, run, s, (jt + kWaves) * kRows, stage ^ 1, jt + kWaves <= qt);
    const char* Ks = base + stage * 2 * kTileBytes;
    const char* Vs = Ks + kTileBytes;
    f32x4 sc[2][2] = {{zero4(), zero4()}, {zero4(), zero4()}}, dp[2][2] = {{zero4(), zero4()}, {zero4(), zero4()}};
    products(sc, Ks, lo, qf, [&](int k) { ring.pair(k); });
    products(dp, Vs, lo, gf, [&](int k) { ring.pair(4 + k); });
    bf16x8 ds[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float p = __builtin_amdgcn_exp2f(fmaf(sc[kb][qb][e], c2, -lse2[qb]));
          if (jt == qt && 16 * kb + 4 * q4 + e > c16 + 16 * qb) p = 0.f;
          dp[kb][qb][e] = p * (dp[kb][qb][e] - delta[qb]);
        }
      ds[qb] = pack8(dp[0][qb], dp[1][qb]);
    }
    accumulate(dq, Ks, lo, ds);
  }
  __syncthreads();   // the rings are done with
  float* blocks = reinterpret_cast<float*>(smem);
  put_block(blocks + w * kBlockFloats, dq, lane);
  __syncthreads();
  const float scale[kWaves] = {a.scale, a.scale, a.scale, a.scale};
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int row = 16 * pass + (tid >> 4), c = tid & 15;
    if (i0 + row >= run.len) break;
    const int t = token_of(run.p0 + i0 + row, s, a.N);
    f32x4 x[2];
    sum_blocks(x, blocks, row, c, scale);
    *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(a.dq) + row_off(a.sdq, at.b, t, at.h) + 8 * c) = pack8(x[0], x[1]);
  }
}

__global__ void __launch_bounds__(64 * kWaves, 1)
bwd_small_kernel(KArgs a, int n_kv, int T, Deal deal_kv, Deal deal_q, int first_block) {
  __shared__ __attribute__((aligned(1024))) char smem[kSmemBwd];
  fetch_args(a, deal_q);
  const int block = first_block + block_id();
  if (block < n_kv)
    dkdv_small_block(a, smem, block, T, deal_kv);
  else
    dq_small_block(a, smem, block - n_kv, T, deal_q);
}

}  // namespace

static long long small_blocks(const KArgs& a) { return (long long)a.B * a.H * a.NG * ragged_tiles(a, kRows); }

// Up to as many workgroups of 32 rows as there are CUs (fewer than eight sequences keep to as many XCDs), for the
// workgroups of 128 (256) rows share a tile between four (eight)
// waves and so need a quarter of the loads once the chip is full; and not for chains so long that these are
// the faster loop.  Forward, us, workgroups of 128 or 256 rows and here: H = 4, groups of 256, N = 1024 (128
// workgroups of 32 rows): 8.6 and 7.1; groups of 2048, N = 2048 (256): 45.7 and 29.7; groups of 4096, H = 2,
// N = 4096 (256): 85 and 95; groups of 512, N = 2560 (320): 13.2 and 14.3.  Short chains take the time of a second round
// badly, so up to eight workgroups to a sequence the busiest XCD has to hold all of its own at once (groups of 96:
// ten sequences of an XCD, 30 workgroups, 6.8 and 5.9; eleven, 33, 6.8 and 9.6; of 192: five 9.0 and 7.2, six, 36, 8.9
// and 9.8; of 288: four, 36, 10.9 and 10.0).
bool fwd_is_small(const KArgs& a) {
  const int T = ragged_tiles(a, kRows);
  return a.D == 128 && a.G <= 2048 && small_blocks(a) <= 256 && (T >= 9 || most_of_an_xcd(a.B * a.H * a.NG) * T <= 32);
}
// Backward (delta and both gradients): groups of 256, N = 1024, H = 4, Hkv = 2 (128) 20.5 and 16.3; H = Hkv = 8 (256)
// 17.9 and 18.5; Hkv = 2 (256) 32.9 and 24.9; groups of 1024, N = 1024, H = 8 (256) 41.4 and 31.4; groups of 2048,
// H = 2, N = 2048 (128) 74.7 and 79.5; groups of 640, N = 2560, H = 4 (320) 25.8 and 31.5; groups of 64,
// N = 1024, H = 8, Hkv = 4 (256) 11.8 and 14.0.
// One workgroup to a CU, and dK/dV's are as many as dQ's where a part is one head: both of the busiest XCD together then
// want to fit into one round of its 32 CUs, a little more as the chains grow, two rounds from ten workgroups to a
// sequence on.  One head to a kv head, sequences of an XCD and the workgroups of both: groups of 96 five (30) 12.2 and
// 9.9, six (36) 11.9 and 13.8; of 128 three (24) 12.3 and 10.1, six (48) 12.6 and 15.7; of 192 three (36) 14.4 and 14.1,
// four (48) 14.4 and 15.7; of 256 two (32) 16.5 and 12.0, three (48) 17.7 and 16.8, four (64) 17 and 18.5; of 320 two (40)
// 17 and 15.5, three (60) 18 and 20; of 512 two (64) 24.3 and 22.7; of 768 one (48) 32 and 21.5, two (96) 32.4 and 38.2.
// With partials, which the others write too: groups of 66 six (36) 15.9 and 15.8, eight (48) 16.8 and 18.3; of 160 four
// (40) 21.0 and 19.2, five (50) 21.2 and 20.1; of 192 four (48) 20.8 and 20.1, six (72) 22.2 and 27.7; of 640 two (80) 32.5
// and 35.8.
bool bwd_is_small(const KArgs& a) {
  const int most = a.G <= 64 ? 128 : a.r > 1 || a.G >= 512 ? 256 : 160;
  if (a.D != 128 || a.G > 1536 || small_blocks(a) > most) return false;
  const int T = ragged_tiles(a, kRows);
  const int dq = most_of_an_xcd(a.B * a.H * a.NG), dkdv = most_of_an_xcd(a.B * a.Hkv * a.NG * a.parts);
  const bool one_head = a.Hkv * a.parts >= a.H;   // to a part
  const int fit = T >= 10 ? 64 : a.parts > 1 ? (T < 4 ? 36 : T < 5 ? 40 : 50) : T < 6 ? 32 : T < 7 ? 36 : 48;
  return !one_head || dq == 1 || (dq + dkdv) * T <= fit;
}

int launch_fwd_small(const KArgs& a, hipStream_t st) {
  const int T = ragged_tiles(a, kRows);
  const Grid g = grid_of(T, a.B * a.H * a.NG, a.r, 32);
  return launch_blocks(fwd_small_kernel, g.blocks, 64 * kWaves, st, a, T, g.deal);
}

int launch_bwd_small(const KArgs& a, bool dq_last, hipStream_t st) {
  const int T = ragged_tiles(a, kRows);
  const Grid kv = grid_of(T, a.B * a.Hkv * a.NG * a.parts, 1, 32), q = grid_of(T, a.B * a.H * a.NG, a.r, 32);
  const int n_first = dq_last ? kv.blocks : kv.blocks + q.blocks;
  const int rc = launch_blocks(bwd_small_kernel, n_first, 64 * kWaves, st, a, kv.blocks, T, kv.deal, q.deal);
  if (rc != 0 || !dq_last) return rc;
  return launch_blocks(bwd_small_kernel, q.blocks, 64 * kWaves, st, a, 0, T, kv.deal, q.deal);
}

}  // namespace s2
