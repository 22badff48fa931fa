// bf16 S2-Attn backward for gfx950, dQ kernel: recomputes P = exp(scale*S - lse) from the stored
// log-sum-exp and uses the softmax-Jacobian form dS = P * (dP - delta), delta_i = dO_i . O_i
// (computed by the pre-pass).  The shift/group map of LongLoRA Algorithm 1 is row addressing only.
//
// A workgroup of WAVES waves owns 32 query rows per wave (128 or 256;  Q^T and dO^T fragments in registers) and walks the
// 64-key tiles up to the diagonal: S^T = K Q^T, dP^T = V dO^T, dQ^T += K^T dS^T with K^T through
// transposing LDS loads.
#pragma once
#include <type_traits>

#include "s2attn_bf16_common.h"
#include "s2attn_device.h"
#include "s2attn_launch.h"

namespace s2 {
namespace {

constexpr int BN = 64;                       // keys per tile
constexpr int kTileBytes = BN * kRowBytes;   // 16 KB

// One 64-key tile of the dQ kernel as 12 steps of 4 MFMAs, each fed by 4 fragments:
//   steps 0-3 / 4-7: S^T and dP^T of key block 0 / 1 over d = 32j .. 32j+31
//   steps 8-11:      dQ^T += K^T dS^T for keys 16k .. 16k+15
// Every step first issues the LDS reads of the next step into the other fragment buffer
// (also across the exp/multiply sections), then runs its own four MFMAs.
// XTR: the transposed fragments' addresses are made of one, tr0 (that of column block 0): a column block
// is bits 6 and 7 of the chunk's offset under the swizzle, eight rows further on flips bit 5 of it.
template <int STEP, bool XTR>
__device__ __forceinline__ void dq_load(bf16x8 (&buf)[4], const char* Ks, const char* Vs, const LaneOffsets& lo,
                                        uint32_t tr0) {
  if constexpr (STEP < 8) {
    constexpr int ROW0 = 32 * (STEP / 4), J = STEP % 4;
    buf[0] = frag_rm<ROW0>(Ks, lo, 2 * J);
    buf[1] = frag_rm<ROW0>(Vs, lo, 2 * J);
    buf[2] = frag_rm<ROW0>(Ks, lo, 2 * J + 1);
    buf[3] = frag_rm<ROW0>(Vs, lo, 2 * J + 1);
  } else if constexpr (XTR) {
    constexpr int ROW0 = 16 * (STEP - 8);
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(S2_LDS(bf16x4, (tr0 ^ (db << 6)) + ROW0 * kRowBytes));
      const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(S2_LDS(bf16x4, (tr0 ^ (db << 6 | 32)) + (ROW0 + 8) * kRowBytes));
      buf[db] = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  } else {
#pragma unroll
    for (int db = 0; db < 4; ++db) buf[db] = frag_tr<16 * (STEP - 8)>(Ks, lo, db);
  }
}

template <int STEP>
__device__ __forceinline__ void dq_mma(const bf16x8 (&buf)[4], const bf16x8 (&qf)[8], const bf16x8 (&dof)[8],
                                       f32x16& sa, f32x16& pa, const bf16x8 (&dsf)[4], f32x16 (&dq_acc)[4]) {
  if constexpr (STEP < 8) {
    constexpr int J = STEP % 4;
    sa = mfma32(buf[0], qf[2 * J], sa);
    pa = mfma32(buf[1], dof[2 * J], pa);
    sa = mfma32(buf[2], qf[2 * J + 1], sa);
    pa = mfma32(buf[3], dof[2 * J + 1], pa);
  } else {
#pragma unroll
    for (int db = 0; db < 4; ++db) dq_acc[db] = mfma32(buf[db], dsf[STEP - 8], dq_acc[db]);
  }
}

// dS^T = P^T * (dP^T - delta) of one 32-key block, packed as two B operands.
template <int ROW0>
__device__ __forceinline__ void dq_ds(f32x16& sa, const f32x16& pa, bf16x8& ds_lo, bf16x8& ds_hi, int j0, int qrow,
                                      float c2, float lse2, float delta, int g32, bool masked) {
  if (masked) {   // wave-uniform: exp2(-inf) = 0 removes keys after the query
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = j0 + ROW0 + 8 * (v >> 2) + 4 * g32 + (v & 3);
      if (key > qrow) sa[v] = -INFINITY;
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) sa[v] = __builtin_amdgcn_exp2f(fmaf(sa[v], c2, -lse2)) * (pa[v] - delta);
  ds_lo = pack8(sa[0], sa[1], sa[2], sa[3], sa[4], sa[5], sa[6], sa[7]);
  ds_hi = pack8(sa[8], sa[9], sa[10], sa[11], sa[12], sa[13], sa[14], sa[15]);
}

template <bool XTR>
__device__ __forceinline__ void dq_tile(f32x16 (&dq_acc)[4], const bf16x8 (&qf)[8], const bf16x8 (&dof)[8],
                                        const char* Ks, const char* Vs, const LaneOffsets& lo, int j0,
                                        int qrow, float c2, float lse2, float delta, int g32, bool masked) {
#define S2_DQ_STEP(N, CUR, NXT)                                   \
  dq_load<N + 1, XTR>(NXT, Ks, Vs, lo, tr0);                      \
  dq_mma<N>(CUR, qf, dof, sa, pa, dsf, dq_acc);                   \
  __builtin_amdgcn_sched_barrier(0)
  bf16x8 fa[4], fb[4], dsf[4];
  f32x16 sa = zero16(), pa = zero16();
  uint32_t tr0 = 0;
  if constexpr (XTR) {   // hidden from the optimizer, which would keep what is made of it ahead of the loop
    tr0 = (uint32_t)(uintptr_t)S2_LDS(const char, Ks) + lo.tr[0][0];
    asm volatile("" : "+v"(tr0));
  }
  dq_load<0, XTR>(fa, Ks, Vs, lo, tr0);
  __builtin_amdgcn_sched_barrier(0);
  S2_DQ_STEP(0, fa, fb);
  S2_DQ_STEP(1, fb, fa);
  S2_DQ_STEP(2, fa, fb);
  S2_DQ_STEP(3, fb, fa);            // loads step 4 (block 1) before the vector section
  dq_ds<0>(sa, pa, dsf[0], dsf[1], j0, qrow, c2, lse2, delta, g32, masked);
  sa = zero16();
  pa = zero16();
  __builtin_amdgcn_sched_barrier(0);
  S2_DQ_STEP(4, fa, fb);
  S2_DQ_STEP(5, fb, fa);
  S2_DQ_STEP(6, fa, fb);
  S2_DQ_STEP(7, fb, fa);            // loads step 8 (first K^T fragments)
  dq_ds<32>(sa, pa, dsf[2], dsf[3], j0, qrow, c2, lse2, delta, g32, masked);
  __builtin_amdgcn_sched_barrier(0);
  S2_DQ_STEP(8, fa, fb);
  S2_DQ_STEP(9, fb, fa);
  S2_DQ_STEP(10, fa, fb);
  dq_mma<11>(fb, qf, dof, sa, pa, dsf, dq_acc);
#undef S2_DQ_STEP
}

// smem: [2 stages][K,V] tiles, afterwards one 8 KB block per wave.  RAGGED: as in the forward
// kernels, and any tile that runs past the end of a group.
template <bool RAGGED, int WAVES>
__device__ __forceinline__ void dq_workgroup(const KArgs& a, int T, const Deal& deal, int block, int tid, char* smem) {
  constexpr int BM = 32 * WAVES;
  constexpr int kPassRows = 4 * WAVES;   // tile rows that the workgroup stages with one load per wave

  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g32 = lane >> 5, l32 = lane & 31;

  int seq, rank;
  if (!decode_block(block, T, deal, seq, rank)) return;
  const HeadPos at = head_of_seq(a, seq);
  const int gidx = at.g, c = at.c, b = at.b, h = at.h;
  int qt = T - 1 - rank;

  const int s = uni(shift_of_head(a, h));
  Run run{gidx * a.G, a.G};                        // the causal run of this block (see the forward kernel)
  int split = uni(split_of_group(a, gidx, s));
  if constexpr (RAGGED) {
    if (!run_of_tile(a, gidx, s, BM, qt, run)) return;
    run.p0 = uni(run.p0); run.len = uni(run.len);
    split = run.len;
  }
  const int i0 = qt * BM;
  const int qw0 = i0 + w * 32;
  const int qrow = qw0 + l32;
  const int lo_w = uni(qw0 >= split ? split : 0);
  const int jt_first = uni((i0 >= split ? split : 0) / BN);
  const float c2 = a.scale_log2;

  const char* kp = static_cast<const char*>(a.k);
  const char* vp = static_cast<const char*>(a.v);

  bf16x8 qf[8], dof[8];
  float lse2, delta;
  {
    const int tok = run_token(a, run, qrow, s);
    const bf16x8* qsrc = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(a.q) + row_off(a.sq, b, tok, h));
    const bf16x8* dsrc = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(a.dout) + row_off(a.so, b, tok, h));
#pragma unroll
    for (int st = 0; st < 8; ++st) { qf[st] = qsrc[2 * st + g32]; dof[st] = dsrc[2 * st + g32]; }
    const size_t ro = ((size_t)b * a.H + h) * a.N + tok;
    lse2 = a.lse2[ro];
    delta = -a.neg_delta[ro];
  }

  const uint32_t smem_base = lds_addr(smem);
  const uint64_t k_row_bytes = (uint64_t)a.sk.t * 2, v_row_bytes = (uint64_t)a.sv.t * 2;
  const int st_row = 4 * w + (lane >> 4);
  const uint32_t st_chunk = (uint32_t)(((lane & 15) ^ swz(st_row)) << 4);
  // aligned staging: scalar base of the tile's 64-token run plus these per-lane offsets
  const uint32_t k_lane = (uint32_t)(st_row * k_row_bytes) + st_chunk;
  const uint32_t v_lane = (uint32_t)(st_row * v_row_bytes) + st_chunk;
  const uint64_t k_head = uni64(reinterpret_cast<uint64_t>(kp) + row_off(a.sk, b, 0, c) * 2);
  const uint64_t v_head = uni64(reinterpret_cast<uint64_t>(vp) + row_off(a.sv, b, 0, c) * 2);
  auto issue_tile = [&](int jt, int stage) {
    const uint32_t ks = smem_base + stage * 2 * kTileBytes + 4 * w * kRowBytes;
    const int row0 = jt * BN;
    const uint32_t tok0 = (uint32_t)token_of(run.p0 + row0, s, a.N);
    if (RAGGED && (row0 + BN > run.len || (int)tok0 + BN > a.N)) {
      // not 64 consecutive tokens: row by row, rows past the end of the run repeat its last row
#pragma unroll
      for (int p = 0; p < BN / kPassRows; ++p) {
        const int tok = run_token(a, run, row0 + kPassRows * p + st_row, s);
        dma16(kp + row_off(a.sk, b, tok, c) * 2 + st_chunk, ks + kPassRows * p * kRowBytes);
        dma16(vp + row_off(a.sv, b, tok, c) * 2 + st_chunk, ks + kPassRows * p * kRowBytes + kTileBytes);
      }
      return;
    }
    const uint64_t kb = k_head + tok0 * k_row_bytes, vb = v_head + tok0 * v_row_bytes;
#pragma unroll
    for (int p = 0; p < BN / kPassRows; ++p) {
      dma16s(kb + p * kPassRows * k_row_bytes, k_lane, ks + kPassRows * p * kRowBytes);
      dma16s(vb + p * kPassRows * v_row_bytes, v_lane, ks + kPassRows * p * kRowBytes + kTileBytes);
    }
  };

  LaneOffsets lo;
  init_lane_offsets(lo, lane);
  f32x16 dq_acc[4];
#pragma unroll
  for (int db = 0; db < 4; ++db) dq_acc[db] = zero16();

  issue_tile(jt_first, 0);
  const int n_tiles = (RAGGED ? uni((min(i0 + BM, run.len) + BN - 1) / BN) : (i0 + BM) / BN) - jt_first;
  // With four waves the stage is a compile-time constant of the body (the loop is unrolled by the
  // number of stages), so every LDS read is lane offset + immediate; in the kernel that shares its
  // registers with dK/dV that spills.
  auto body = [&](auto stage_c, int n) __attribute__((always_inline)) {
    const int STAGE = stage_c;
    const int jt = jt_first + n;
    wait_vmcnt0();
    __syncthreads();
    if (n + 1 < n_tiles) issue_tile(jt + 1, STAGE ^ 1);
    const int j0 = jt * BN;
    const char* Ks = smem + STAGE * 2 * kTileBytes;
    const char* Vs = Ks + kTileBytes;
    if (j0 > qw0 + 31 || j0 + BN - 1 < lo_w) return;   // wholly outside this wave's visible keys
    dq_tile<RAGGED && WAVES == 8>(dq_acc, qf, dof, Ks, Vs, lo, j0, qrow, c2, lse2, delta, g32, j0 + BN - 1 > qw0);
  };
  if constexpr (WAVES == 4) {
    for (int n = 0; n < n_tiles; n += 2) {
      body(std::integral_constant<int, 0>{}, n);
      if (n + 1 < n_tiles) body(std::integral_constant<int, 1>{}, n + 1);
    }
  } else {
#pragma unroll 1
    for (int n = 0; n < n_tiles; ++n) body(n & 1, n);
  }
  __syncthreads();

  char* region = smem + w * (32 * kRowBytes);
  acc_to_lds(region, dq_acc, a.scale, l32, g32);
  wave_lds_order();
  store_wave_rows<RAGGED>(a, a.dq, a.sdq, region, run, qw0, s, b, h, lane);
}

template <bool RAGGED>
__global__ void __launch_bounds__(256, 2)
bwd_dq_bf16_kernel(KArgs a, int T, Deal deal, int first_block) {
  __shared__ __attribute__((aligned(1024))) char smem[4 * kTileBytes];
  dq_workgroup<RAGGED, 4>(a, T, deal, first_block + block_id(), thread_id(), smem);
}

}  // namespace

}  // namespace s2
