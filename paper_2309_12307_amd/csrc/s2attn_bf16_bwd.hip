// bf16 S2-Attn backward, dK/dV kernel for gfx950 (D = 128), two waves per SIMD ("role split").
//
// A workgroup (8 waves on one CU) owns 128 keys of one (batch, kv head, group) in the rolled
// frame of the kv head's class (LongLoRA Algorithm 1: the shift is row addressing only) and
// walks the 64-row query tiles at or below the diagonal (from the end of the group down to
// the diagonal) for every query head of the kv head, or of one part of them (part_heads).  The four products of the
// softmax-Jacobian backward (dS = P * (dP - delta), P recomputed from the stored
// log-sum-exp) are split between the two waves that share a SIMD and a 32-key block, so that
// each fits in 256 registers with all accumulators in ordinary vector registers:
//   wave A (0-3):  S = Q K^T,  P = exp2(c S - lse2)  ->  LDS (fp32),   dV^T += dO^T P
//   wave B (4-7):  dP - delta = dO V^T - delta,  P <- LDS,  dS = P (dP - delta),  dK^T += Q^T dS
// B finishes tile n-1 (dS, dK) at the start of iteration n, after the barrier that also
// publishes the staged tile n, so the hand-over of P costs no barrier of its own, and the
// two waves of a SIMD alternate between the matrix and the vector unit.  Keys are
// lane-indexed and queries register-indexed in S, dP, P and dS, so P and dS are B operands
// as they come out of the accumulators.  Q tiles live in three LDS stages (B still reads
// Q^T of tile n-1 during iteration n), dO tiles, P and the lse / delta rows in two.
// The two query tiles that touch the diagonal run the same code with a causal mask on P;
// blocks wholly above the diagonal are computed with P = 0 rather than branched around.
#include <type_traits>

#include "s2attn_bf16_common.h"
#include "s2attn_bf16_dq.h"
#include "s2attn_device.h"
#include "s2attn_launch.h"

namespace s2 {
namespace {

constexpr int kQT = 64;                            // query rows per tile
constexpr int kQTBytes = kQT * kRowBytes;          // 16 KB
constexpr int kOffQ = 0;                           // 3 stages of Q
constexpr int kOffdO = 3 * kQTBytes;               // 2 stages of dO
constexpr int kOffP = 5 * kQTBytes;                // 2 buffers x 4 key blocks x 2 query blocks x 4 KB (fp32 P)
constexpr int kPBlockBytes = 4096;
constexpr int kPBufBytes = 4 * 2 * kPBlockBytes;   // 32 KB
constexpr int kOffRows = kOffP + 2 * kPBufBytes;   // [2 stages][lse2, -delta][64] floats
constexpr int kSmemBytes = kOffRows + 2 * 2 * kQT * 4;

// Scores of both 32-query blocks of a tile against this wave's 32 keys: acc0/acc1 +=
// X[block] Bf^T, X = Q (role A) or dO (role B) read row-major from LDS, Bf = the wave's
// K^T or V^T fragments.  Steps of 4 MFMAs; every step first issues the reads of the next.
template <int STEP>
__device__ __forceinline__ void sc_load(bf16x8 (&buf)[4], const char* Xs, const LaneOffsets& lo) {
  buf[0] = frag_rm<0>(Xs, lo, 2 * STEP);
  buf[1] = frag_rm<32>(Xs, lo, 2 * STEP);
  buf[2] = frag_rm<0>(Xs, lo, 2 * STEP + 1);
  buf[3] = frag_rm<32>(Xs, lo, 2 * STEP + 1);
}
template <int STEP>
__device__ __forceinline__ void sc_mma(const bf16x8 (&buf)[4], const bf16x8 (&bf)[8], f32x16& acc0, f32x16& acc1) {
  acc0 = mfma32(buf[0], bf[2 * STEP], acc0);
  acc1 = mfma32(buf[1], bf[2 * STEP], acc1);
  acc0 = mfma32(buf[2], bf[2 * STEP + 1], acc0);
  acc1 = mfma32(buf[3], bf[2 * STEP + 1], acc1);
}
__device__ __forceinline__ void scores(f32x16& acc0, f32x16& acc1, const char* Xs, const LaneOffsets& lo,
                                       const bf16x8 (&bf)[8]) {
  bf16x8 fa[4], fb[4], fc[4];
  sc_load<0>(fa, Xs, lo);
  sc_load<1>(fb, Xs, lo);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(1);   // matrix work goes ahead of the other wave's vector work
  sc_load<2>(fc, Xs, lo); sc_mma<0>(fa, bf, acc0, acc1); __builtin_amdgcn_sched_barrier(0);
  sc_load<3>(fa, Xs, lo); sc_mma<1>(fb, bf, acc0, acc1); __builtin_amdgcn_sched_barrier(0);
  sc_mma<2>(fc, bf, acc0, acc1); __builtin_amdgcn_sched_barrier(0);
  sc_mma<3>(fa, bf, acc0, acc1);
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_sched_barrier(0);
}

// acc^T (128 x 32 keys) += X^T W for the 64 queries of a tile: X^T = dO^T (role A) or Q^T
// (role B) through transposing LDS reads, W = P or dS as four 16-query B operands.
template <int STEP>
__device__ __forceinline__ void ac_load(bf16x8 (&buf)[4], const char* Xs, const LaneOffsets& lo) {
#pragma unroll
  for (int db = 0; db < 4; ++db) buf[db] = frag_tr<16 * STEP>(Xs, lo, db);
}
__device__ __forceinline__ void ac_mma(const bf16x8 (&buf)[4], bf16x8 wf, f32x16 (&acc)[4]) {
#pragma unroll
  for (int db = 0; db < 4; ++db) acc[db] = mfma32(buf[db], wf, acc[db]);
}
// `fa` and `fb` already hold the fragments of steps 0 and 1 (loaded ahead of the vector work).
__device__ __forceinline__ void accumulate(f32x16 (&acc)[4], bf16x8 (&fa)[4], bf16x8 (&fb)[4], const char* Xs,
                                           const LaneOffsets& lo, const bf16x8 (&wf)[4]) {
  bf16x8 fc[4];
  __builtin_amdgcn_s_setprio(1);
  ac_load<2>(fc, Xs, lo); ac_mma(fa, wf[0], acc); __builtin_amdgcn_sched_barrier(0);
  ac_load<3>(fa, Xs, lo); ac_mma(fb, wf[1], acc); __builtin_amdgcn_sched_barrier(0);
  ac_mma(fc, wf[2], acc); __builtin_amdgcn_sched_barrier(0);
  ac_mma(fa, wf[3], acc);
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_sched_barrier(0);
}

// 16 bytes per lane, written through to memory (system scope): the stored dS is not read
// again by this kernel, and left to the L2's default policy it evicts the Q and dO tiles that
// the workgroups of an XCD share (measured: 3.6 times the HBM reads).
__device__ __forceinline__ void store_ds(char* dst, bf16x8 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1" :: "v"(dst), "v"(v) : "memory");
}

// Ahead of the two tile loops: pads the code so that they start at the same address modulo 8 whatever
// stands before them.  Their speed depends on it (most of their instructions are 8 bytes long): with
// one 4-byte instruction more ahead of both, N = 32768, H = 32, G = 8192 went from 4.06 to 4.14 ms and,
// at another phase, N = 16000, H = 32, G = 4000 (partial tiles) from 1.07 to 1.12 ms; as placed here
// both run at the lower figure.
__device__ __forceinline__ void loop_phase() { asm volatile(".p2align 3"); }

// SPILL: role B also stores dS of every tile it finishes (bf16, the operand it feeds to the
// dK product) for the dQ kernel, which then needs neither S nor dP again.
// RAGGED: G is not a multiple of 128, the shift not of 64 or a Variant 2 split not of 128: the last
// tiles of a run may be partial and the wrap point may fall inside a tile.  Such a tile is staged
// row by row; every other tile is 64 consecutive tokens, wherever it starts, and takes the aligned
// path.  N = 100000, H = 32, G = 25000: forward + backward 86.9 ms with a dK/dV kernel of its own for
// these shapes (one wave per SIMD, every row staged by itself) and the four-wave forward, 82.1 ms
// with this one and the eight-wave forward.
template <bool SPILL, bool RAGGED>
__device__ __forceinline__ void dkdv_workgroup(const KArgs& a, int T, const Deal& deal, int block, int tid, char* smem) {
  const int lane = tid & 63, w = uni(tid >> 6);
  const int g32 = lane >> 5, l32 = lane & 31;
  const bool role_b = w >= 4;
  const int kb = w & 3;

  // block -> (batch, kv head, part of its query heads, group, key tile); heaviest key tiles (jt = 0) first
  int seq, jt;
  if (!decode_block(block, T, deal, seq, jt)) return;
  const KvPos at = kv_of_seq(a, seq);
  const int gidx = at.g, c = at.c, b = at.b;
  int h_lo, nheads, s;                               // query heads [h_lo, h_lo + nheads), all of one class
  part_heads(a, c, at.part, h_lo, nheads, s);
  // the causal run of these keys and the query rows [j0, q_end) of it that see them: up to the end
  // of the group, or up to the split for the first block of a split wrap-around group (Variant 2,
  // Appendix B.3).  An aligned split is a multiple of the key tile; a ragged one makes two runs.
  Run run{gidx * a.G, a.G};
  if constexpr (RAGGED) {
    if (!run_of_tile(a, gidx, s, 128, jt, run)) return;
    jt = uni(jt); run.p0 = uni(run.p0); run.len = uni(run.len);
  }
  const int j0 = jt * 128;
  const int kw0 = j0 + 32 * kb;                      // first key of this wave
  const int key = kw0 + l32;
  const int split = uni(split_of_group(a, gidx, s));
  const int q_end = RAGGED ? run.len : (j0 < split ? split : a.G);
  const int nq = uni((q_end - j0 + kQT - 1) / kQT);   // query tiles of one head
  const int n_iter = nheads * nq;
  const float c2 = a.scale_log2;

  // loop-invariant B operand of this wave's 32 keys: K^T (role A) or V^T (role B)
  bf16x8 bfrag[8];
  {
    const int tok = run_token(a, run, key, s);
    const bf16x8* src = reinterpret_cast<const bf16x8*>(
        role_b ? static_cast<const __bf16*>(a.v) + row_off(a.sv, b, tok, c)
               : static_cast<const __bf16*>(a.k) + row_off(a.sk, b, tok, c));
#pragma unroll
    for (int st = 0; st < 8; ++st) bfrag[st] = src[2 * st + g32];
  }

  // staging: wave w fills tile rows 4w .. 4w+3 and 32+4w .. 32+4w+3 of Q and of dO; a tile is
  // one contiguous run of 64 tokens: scalar base + fixed per-lane offset
  const uint32_t smem_base = lds_addr(smem);
  const uint64_t q_row_bytes = (uint64_t)a.sq.t * 2, do_row_bytes = (uint64_t)a.so.t * 2;
  const int st_row = 4 * w + (lane >> 4);
  const uint32_t st_chunk = (uint32_t)(((lane & 15) ^ swz(st_row)) << 4);
  const uint32_t q_lane = (uint32_t)(st_row * q_row_bytes) + st_chunk;
  const uint32_t do_lane = (uint32_t)(st_row * do_row_bytes) + st_chunk;
  const uint64_t q_batch = uni64(reinterpret_cast<uint64_t>(a.q) + (uint64_t)b * a.sq.b * 2);
  const uint64_t do_batch = uni64(reinterpret_cast<uint64_t>(a.dout) + (uint64_t)b * a.so.b * 2);
  // tile (hh, it) of the flattened sequence n = hh * nq + it; q_stage = n mod 3, o_stage = n mod 2
  auto issue_tile = [&](int hh, int it, int q_stage, int o_stage) {
    const int h = h_lo + hh;
    const int row0 = j0 + it * kQT;
    const uint32_t tok0 = (uint32_t)token_of(run.p0 + row0, s, a.N);
    const uint32_t qs = smem_base + kOffQ + q_stage * kQTBytes + 4 * w * kRowBytes;
    const uint32_t dos = smem_base + kOffdO + o_stage * kQTBytes + 4 * w * kRowBytes;
    const uint32_t rows_dst = smem_base + kOffRows + ((o_stage * 2 + w) * kQT) * 4;
    if (RAGGED && (row0 + kQT > run.len || (int)tok0 + kQT > a.N)) {
      // rows past the end of the run repeat its last row; their P is set to zero
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int tok = run_token(a, run, row0 + 32 * p + st_row, s);
        dma16(static_cast<const char*>(a.q) + row_off(a.sq, b, tok, h) * 2 + st_chunk, qs + 32 * p * kRowBytes);
        dma16(static_cast<const char*>(a.dout) + row_off(a.so, b, tok, h) * 2 + st_chunk, dos + 32 * p * kRowBytes);
      }
      if (w < 2)
        dma4((w == 0 ? a.lse2 : a.neg_delta) + ((size_t)b * a.H + h) * a.N + run_token(a, run, row0 + lane, s), rows_dst);
      return;
    }
    const uint64_t qb = uni64(q_batch + tok0 * q_row_bytes + (uint64_t)h * a.sq.h * 2);
    const uint64_t dob = uni64(do_batch + tok0 * do_row_bytes + (uint64_t)h * a.so.h * 2);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      dma16s(qb + p * 32 * q_row_bytes, q_lane, qs + 32 * p * kRowBytes);
      dma16s(dob + p * 32 * do_row_bytes, do_lane, dos + 32 * p * kRowBytes);
    }
    if (w < 2) {   // wave 0: lse * log2(e), wave 1: -delta; 64 rows each
      const uint64_t ro = (((uint64_t)b * a.H + h) * a.N + tok0) * 4;
      dma4s(uni64(reinterpret_cast<uint64_t>(w == 0 ? a.lse2 : a.neg_delta) + ro), lane * 4, rows_dst);
    }
  };

  LaneOffsets lo;
  init_lane_offsets(lo, lane);
  f32x16 acc[4];                  // dV^T (role A) or dK^T (role B) of this wave's keys
#pragma unroll
  for (int db = 0; db < 4; ++db) acc[db] = zero16();

  // The flattened tile sequence n = 0 .. n_iter - 1 runs over the query tiles from the end of
  // the group down to the diagonal, all query heads of a tile one after the other.  Every
  // workgroup of a (kv head, group) starts at the last query tile whatever its key tile, so the
  // workgroups that run together read the same Q and dO tile at about the same time and the
  // tile is fetched from HBM once.  (From the diagonal upwards and head by head the
  // workgroups are spread over a window of tiles and, with r heads per kv head, drift apart
  // over r heads' worth of Q and dO: at r = 8 the kernel then reads 8 times as much from HBM
  // and takes 7 % longer; at r = 1 it is 2 % slower.)
  auto advance = [&](int& hh, int& it) {
    if (++hh == nheads) { hh = 0; --it; }
  };
  const int it_first = nq - 1;
  int hh_next = 0, it_next = it_first;     // tile n + 1 (to be staged)
  if (n_iter > 0) issue_tile(0, it_first, 0, 0);   // (a part may be empty)
  advance(hh_next, it_next);

  if (!role_b) {
    // ------------------------------------------------------------------ role A
    int hh_cur = 0, it = it_first;    // tile n
    int q_st = 0;                     // n mod 3
    int n = 0;
    loop_phase();
    do {
      const int o_st = n & 1;
      wait_vmcnt0();        // this wave's part of tile n has landed
      __syncthreads();      // tile n is complete; everyone has left iteration n-1
      if (n + 1 < n_iter) {
        issue_tile(hh_next, it_next, q_st == 2 ? 0 : q_st + 1, o_st ^ 1);
        advance(hh_next, it_next);
      }
      if (n < n_iter) {
        const char* Qs = smem + kOffQ + q_st * kQTBytes;
        const char* dOs = smem + kOffdO + o_st * kQTBytes;
        const float* lse2_s = reinterpret_cast<const float*>(smem + kOffRows) + (o_st * 2) * kQT;
        char* Px = smem + kOffP + o_st * kPBufBytes + kb * 2 * kPBlockBytes + lane * 16;
        const int q0 = j0 + it * kQT;
        // tiles 0 and 1 touch the diagonal of the 128 keys, a partial last tile holds padding rows
        const bool masked = it < 2 || (RAGGED && q0 + kQT > run.len);
        // lse rows of both blocks (queries are register-indexed: 16 values per block and lane
        // half), fetched ahead of the scores so that the vector work below never waits on LDS
        float4 lr[2][4];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int vv = 0; vv < 4; ++vv)
            lr[mb][vv] = *reinterpret_cast<const float4*>(lse2_s + 32 * mb + 8 * vv + 4 * g32);
        f32x16 s0 = zero16(), s1 = zero16();
        scores(s0, s1, Qs, lo, bfrag);
        bf16x8 fa[4], fb[4];
        ac_load<0>(fa, dOs, lo);       // first dO^T fragments arrive during the vector work
        ac_load<1>(fb, dOs, lo);
        bf16x8 pf[4];
        auto softmax_block = [&](auto masked_c, int mb, f32x16& sx) {
          constexpr bool MASKED = decltype(masked_c)::value;
#pragma unroll
          for (int vv = 0; vv < 4; ++vv) {
            const float ls[4] = {lr[mb][vv].x, lr[mb][vv].y, lr[mb][vv].z, lr[mb][vv].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float p = __builtin_amdgcn_exp2f(fmaf(sx[4 * vv + e], c2, -ls[e]));
              if constexpr (MASKED) {
                const int row = q0 + 32 * mb + 8 * vv + 4 * g32 + e;
                if (key > row || (RAGGED && row >= run.len)) p = 0.f;
              }
              sx[4 * vv + e] = p;
            }
            *reinterpret_cast<float4*>(Px + mb * kPBlockBytes + vv * 1024) =
                make_float4(sx[4 * vv], sx[4 * vv + 1], sx[4 * vv + 2], sx[4 * vv + 3]);
          }
          pf[2 * mb] = pack8(sx[0], sx[1], sx[2], sx[3], sx[4], sx[5], sx[6], sx[7]);
          pf[2 * mb + 1] = pack8(sx[8], sx[9], sx[10], sx[11], sx[12], sx[13], sx[14], sx[15]);
        };
        if (masked) {
          softmax_block(std::true_type{}, 0, s0);
          softmax_block(std::true_type{}, 1, s1);
        } else {
          softmax_block(std::false_type{}, 0, s0);
          softmax_block(std::false_type{}, 1, s1);
        }
        __builtin_amdgcn_sched_barrier(0);
        accumulate(acc, fa, fb, dOs, lo, pf);
      }
      advance(hh_cur, it);
      q_st = q_st == 2 ? 0 : q_st + 1;
    } while (++n <= n_iter);
  } else {
    // ------------------------------------------------------------------ role B
    int q_st = 0;                     // n mod 3
    f32x16 dp0 = zero16(), dp1 = zero16();   // dP - delta of the pending tile
    // dS blobs of this workgroup: those of key tile jt of head h_lo, one after the other along
    // the query tiles; the next head's are a whole (head, group-count) block further on
    char* ds_lane = nullptr;
    long long ds_head_stride = 0;
    int hh_prev = 0, it_prev = 0;     // tile n - 1 (valid from n = 1 on)
    int hh_cur = 0, it_cur = it_first;   // tile n
    if constexpr (SPILL) {
      const long long per_group = ds_blobs_per_group(T);
      const long long first = ((long long)(b * a.c_count * a.r + (h_lo - a.c_begin * a.r)) * a.NG + gidx) * per_group +
                              ds_blob_index(T, jt, 0);
      ds_lane = static_cast<char*>(a.ds_spill) + first * kDsBlobBytes + kb * 4096 + lane * 16;
      ds_head_stride = (long long)a.NG * per_group * kDsBlobBytes;
    }
    int n = 0;
    loop_phase();
    do {
      const int o_st = n & 1;
      wait_vmcnt0();
      __syncthreads();      // also publishes the P of tile n-1
      if (n + 1 < n_iter) {
        issue_tile(hh_next, it_next, q_st == 2 ? 0 : q_st + 1, o_st ^ 1);
        advance(hh_next, it_next);
      }
      const bool has_prev = n >= 1, has_cur = n < n_iter;
      const char* Qs = smem + kOffQ + (q_st == 0 ? 2 : q_st - 1) * kQTBytes;   // tile n-1
      bf16x8 fa[4], fb[4], dsf[4];
      if (has_prev) {
        // finish tile n-1: dS = P * (dP - delta)
        const char* Px = smem + kOffP + (o_st ^ 1) * kPBufBytes + kb * 2 * kPBlockBytes + lane * 16;
        float4 pr[2][4];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int vv = 0; vv < 4; ++vv)
            pr[mb][vv] = *reinterpret_cast<const float4*>(Px + mb * kPBlockBytes + vv * 1024);
        ac_load<0>(fa, Qs, lo);
        ac_load<1>(fb, Qs, lo);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
          f32x16& dx = mb == 0 ? dp0 : dp1;
#pragma unroll
          for (int vv = 0; vv < 4; ++vv) {
            const float4 p4 = pr[mb][vv];
            dx[4 * vv + 0] = p4.x * dx[4 * vv + 0];
            dx[4 * vv + 1] = p4.y * dx[4 * vv + 1];
            dx[4 * vv + 2] = p4.z * dx[4 * vv + 2];
            dx[4 * vv + 3] = p4.w * dx[4 * vv + 3];
          }
          dsf[2 * mb] = pack8(dx[0], dx[1], dx[2], dx[3], dx[4], dx[5], dx[6], dx[7]);
          dsf[2 * mb + 1] = pack8(dx[8], dx[9], dx[10], dx[11], dx[12], dx[13], dx[14], dx[15]);
        }
        if constexpr (SPILL) {
          // the four packed operands as they are: each store is 1 KB of consecutive bytes
          char* dst = ds_lane + hh_prev * ds_head_stride + (long long)it_prev * kDsBlobBytes;
#pragma unroll
          for (int f = 0; f < 4; ++f)
            store_ds(dst + 1024 * f, dsf[f]);
        }
      }
      if constexpr (SPILL) {   // tile n becomes tile n - 1
        hh_prev = hh_cur; it_prev = it_cur;
        advance(hh_cur, it_cur);
      }
      if (has_cur) {
        // dP - delta of tile n: the accumulators start at -delta (per query row = per register);
        // the rows are fetched here so that they arrive during the matrix work below
        const float* nd_s = reinterpret_cast<const float*>(smem + kOffRows) + (o_st * 2 + 1) * kQT;
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) {
          const float4 d0 = *reinterpret_cast<const float4*>(nd_s + 8 * vv + 4 * g32);
          const float4 d1 = *reinterpret_cast<const float4*>(nd_s + 32 + 8 * vv + 4 * g32);
          dp0[4 * vv] = d0.x; dp0[4 * vv + 1] = d0.y; dp0[4 * vv + 2] = d0.z; dp0[4 * vv + 3] = d0.w;
          dp1[4 * vv] = d1.x; dp1[4 * vv + 1] = d1.y; dp1[4 * vv + 2] = d1.z; dp1[4 * vv + 3] = d1.w;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (has_prev) accumulate(acc, fa, fb, Qs, lo, dsf);   // dK^T += Q^T dS
      if (has_cur) scores(dp0, dp1, smem + kOffdO + o_st * kQTBytes, lo, bfrag);
      q_st = q_st == 2 ? 0 : q_st + 1;
    } while (++n <= n_iter);
  }
  if (a.dkv_partial) {   // contiguous fp32 partial of this part, summed by the combine pass
    const size_t elems = (size_t)a.B * a.N * a.Hkv * 128;
    if (RAGGED && key >= run.len) return;   // padding key of a partial tile
    const int tok = token_of(run.p0 + key, s, a.N);
    float* dst = a.dkv_partial + (size_t)((role_b ? 0 : a.parts) + at.part) * elems +
                 ((size_t)((size_t)b * a.N + tok) * a.Hkv + c) * 128 + 4 * g32;
    const float mul = role_b ? a.scale : 1.f;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int vv = 0; vv < 4; ++vv)
        *reinterpret_cast<float4*>(dst + 32 * db + 8 * vv) =
            make_float4(acc[db][4 * vv] * mul, acc[db][4 * vv + 1] * mul, acc[db][4 * vv + 2] * mul, acc[db][4 * vv + 3] * mul);
    return;
  }

  // ---- store this wave's 32 x 128 block (dV for role A, dK for role B) at un-rolled rows, turned
  // through LDS that nobody else touches after the barrier of the last iteration, so that no
  // further barrier is needed and A stores dV while B still works on the last tile: A the dO
  // stages (read up to iteration n_iter - 1), B its part of the P buffer that this iteration's A
  // would have filled.
  // What a workgroup does before its first and after its last tile is a sixth of its time at
  // G = 2048: this, V without the sign it was once loaded with and the set-up moved ahead of the
  // wait for the key fragments take 1.4 % off forward + backward at N = 8192, H = 32, G = 2048.
  static_assert(2 * kQTBytes == 4 * 32 * kRowBytes && 2 * kPBlockBytes == 32 * kRowBytes, "one block per wave");
  char* region = smem + (role_b ? kOffP + (n_iter & 1) * kPBufBytes : kOffdO) + kb * (32 * kRowBytes);
  acc_to_lds(region, acc, role_b ? a.scale : 1.f, l32, g32);
  wave_lds_order();
  store_wave_rows<RAGGED>(a, role_b ? a.dk : a.dv, role_b ? a.sdk : a.sdv, region, run, kw0, s, b, c, lane);
}

template <bool SPILL, bool RAGGED>
__global__ void __launch_bounds__(512, 1)
bwd_dkdv_split_kernel(KArgs a, int T, Deal deal, int first_block) {
  __shared__ __attribute__((aligned(1024))) char smem[kSmemBytes];
  dkdv_workgroup<SPILL, RAGGED>(a, T, deal, first_block + block_id(), thread_id(), smem);
}

// Both in one launch (kv_first: dK/dV first): neither needs the other, and where one of them does not
// fill the chip their chains of tiles run side by side.  dQ takes workgroups of eight waves here.
template <bool RAGGED>
__global__ void __launch_bounds__(512, 1)
bwd_both_kernel(KArgs a, int n_first, int kv_first, int T_kv, Deal deal_kv, int T_q, Deal deal_q) {
  __shared__ __attribute__((aligned(1024))) char smem[kSmemBytes];
  if constexpr (!RAGGED) fetch_args(a, deal_q);   // (partial tiles: 3 % slower with it, no registers left)
  const int id = block_id();
  const bool first = id < n_first;
  const int block = first ? id : id - n_first;
  // the thread index is hidden from the optimizer in each branch: it otherwise computes what the two
  // have in common ahead of the branch, and spills what it then has to keep
  int tid = thread_id();
  if (__builtin_expect(first != (kv_first != 0), 0)) {
    asm volatile("" : "+v"(tid));
    dq_workgroup<RAGGED, 8>(a, T_q, deal_q, block, tid, smem);
    return;
  }
  dkdv_workgroup<false, RAGGED>(a, T_kv, deal_kv, block, thread_id(), smem);
}

}  // namespace

static int bwd_launched() { return hipGetLastError() == hipSuccess ? 0 : -1; }

int launch_bwd_dkdv_bf16(const KArgs& a, hipStream_t st) {
  if (a.D == 64) return launch_bwd_dkdv_d64(a, st);
  const int T = a.ragged ? ragged_tiles(a, 128) : a.G / 128;
  const Grid g = grid_of(T, a.B * a.c_count * a.NG * a.parts, 1, 32);   // 32 CUs per XCD, one workgroup each
  if (a.ds_spill) return launch_blocks(bwd_dkdv_split_kernel<true, false>, g.blocks, 512, st, a, T, g.deal);
  if (a.ragged) return launch_blocks(bwd_dkdv_split_kernel<false, true>, g.blocks, 512, st, a, T, g.deal);
  return launch_blocks(bwd_dkdv_split_kernel<false, false>, g.blocks, 512, st, a, T, g.deal);
}

int launch_bwd_dq_bf16(const KArgs& a, hipStream_t st) {
  if (a.D == 64) return launch_bwd_dq_d64(a, st);
  const int T = a.ragged ? ragged_tiles(a, 128) : a.G / 128;
  const Grid g = grid_of(T, a.B * a.H * a.NG, a.r, 64);                 // 32 CUs per XCD, two workgroups each
  if (a.ragged) return launch_blocks(bwd_dq_bf16_kernel<true>, g.blocks, 256, st, a, T, g.deal);
  return launch_blocks(bwd_dq_bf16_kernel<false>, g.blocks, 256, st, a, T, g.deal);
}

// dK/dV and dQ in one launch where that is faster; 1: not for this shape, launch them one by one.
// Up to six workgroups per CU: the chip is not full, or a good part of the time goes into the tails
// of the two launches, which here lie beside each other.  Backward, us, one by one and in one launch: H = 8, N = 2048,
// G = 256 26.2 and 18.6; N = 4096, G = 1024 62.0 and 45.9; H = 32, Hkv = 1, N = 8192 513 and 500; H = 8, N = 16384 (1536
// workgroups) 482 and 466.  With more workgroups
// nothing is gained (H = 32, N = 8192, 3072 workgroups: 719 and 719) or lost to the eight-wave
// dQ (H = 64, Hkv = 8, N = 32768: 18.25 and 18.70 ms).
// Groups of 128 and less leave half or more of dQ's 256 rows empty, so they share a launch only up to 700
// workgroups, with long chains of dK/dV beside them (8 query heads to a kv head, 16) up to 1100 or the same
// 1536.  Backward, G = 128: H = 8, N = 2048 (256 workgroups) 14.6 us in one launch and 20.7; H = 32, Hkv = 8,
// N = 2048 (640) 38.6 and 40.2, N = 4096 (1280) 75.4 and 62.2; H = 4, Hkv = 2, N = 16384 (768) 44.1 and 38.0;
// Hkv = H / 8: H = 8, N = 2048 (576) 42.5 and 50.9, G = 64, N = 2048 (1152) 43.6 and 42.6; H = 32, Hkv = 1,
// G = 100, N = 4000 (1360) 86 and 109.
// The kernel with the longer chains goes first, so that short ones fill the end: a 64-key tile of
// dQ's 256 rows is half as much work again as a 64-row tile of dK/dV's 128 keys, of which there is
// one for every query head of the part (H = 8, N = 4096: 77.2 us with dK/dV first).
int launch_bwd_both_bf16(const KArgs& a, hipStream_t st) {
  if (a.D == 64) return launch_bwd_both_d64(a, st);
  const bool partial = a.ragged || a.G % 256 != 0 || (a.split < a.G && a.split % 256 != 0);
  const int T_kv = partial ? ragged_tiles(a, 128) : a.G / 128, T_q = partial ? ragged_tiles(a, 256) : a.G / 256;
  const Grid kv = grid_of(T_kv, a.B * a.Hkv * a.NG * a.parts, 1, 32);
  const Grid q = grid_of(T_q, a.B * a.H * a.NG, a.r, 32);
  // counted with the padding of the XCDs and of the last walks (7 % of a grid in the mean, 16 % in one of ten)
  if (kv.blocks + q.blocks > kOneLaunchBlocks) return 1;
  if (a.G <= 128 && a.r < 16 && a.B * a.NG * (a.Hkv * a.parts * T_kv + a.H * T_q) > (a.r < 8 ? 700 : 1100)) return 1;
  const int kv_first = 2 * a.r >= 3 * a.parts;
  const int n_first = kv_first ? kv.blocks : q.blocks;
  if (partial)
    hipLaunchKernelGGL(bwd_both_kernel<true>, dim3(kv.blocks + q.blocks), dim3(512), 0, st, a,
                       n_first, kv_first, T_kv, kv.deal, T_q, q.deal);
  else
    hipLaunchKernelGGL(bwd_both_kernel<false>, dim3(kv.blocks + q.blocks), dim3(512), 0, st, a,
                       n_first, kv_first, T_kv, kv.deal, T_q, q.deal);
  return bwd_launched();
}

}  // namespace s2
