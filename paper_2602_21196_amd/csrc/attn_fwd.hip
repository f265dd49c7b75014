// Causal GQA flash-attention forward for gfx950.
//
// Computes, for each query row i of each head of the chunk, the softmax of
// the scaled scores q_i.k_j/sqrt(d) over the visible keys and its weighted
// sum of values (paper Section 2.1), plus the row log-sum-exp (Section 2.3,
// "the final log-sum-exponent").  Online softmax over key stages keeps HBM
// traffic at O(S d) per head.
//
// Q, K, V and O are read and written where the caller has them (any row and
// head stride): one launch covers all heads of all sequences of a call, with
// no packing.  Against one launch per chunk between pack, merge and unpack
// kernels: 8192 tokens, 4 heads, one head a chunk 408 -> 86 us (12 % -> 58 % of
// 1378 TFLOP/s, an 8192^3 product's rate); 131072 tokens unchanged.
//
// Work decomposition
//   workgroup = 8 waves of 32 query rows x a part of every stage's keys: 256
//               rows x 128 keys, 128 x 64 or 64 x 32 (attn_fwd_key_parts), one
//               query block of one head (two waves per SIMD, one workgroup per
//               CU); the parts of a row are folded in fp32 through LDS.  Up to
//               128 queries on more than 8192 keys: two workgroups, a half of
//               the keys each (attn_fwd_half_stage)
//   key stage = 128 keys, double-buffered in LDS (K rows 32 KB, V rows 32 KB),
//               filled by buffer->LDS copies issued one stage ahead
//   per wave per stage: S^T = K . Q^T    (4 x 8 MFMA 32x32x16, keys on rows)
//                       O^T += V^T . P^T (8 x 4 MFMA), or a half or a quarter
// Computing S^T (keys x queries) puts one query column in each lane: the
// scores of a row sit in one lane pair, and the C tile converts in registers
// into the B operand of the P.V product, whose V^T operand is read out of
// the V rows with transposing LDS reads (tr_operand, common.h).  A stage of
// 128 keys per barrier halves the copies and barriers per product against
// 64-key tiles, and 256 rows per workgroup halve the L2->LDS traffic per
// query against 128.
//
// Lazy rescaling: probabilities are taken against a reference max m_ref that
// moves only when needed.  A lane's sum of its stage probabilities bounds
// each of them, so the row max is computed only when that sum exceeds 2^8 (or
// is not a number, as on the first stage); O = acc / l and lse = m_ref + log l
// are exact for any reference.  Row sums add the bf16-rounded probabilities
// that enter the P.V product (v_dot2_f32_bf16), so O is normalised by the
// weights it was built from.  Query blocks are dispatched longest-first.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace upipe {

namespace {

constexpr int BKS = 128;       // keys per LDS stage
constexpr int K_TILE = BKS * HEAD_DIM * 2;       // [128][128] bf16 = 32 KB
constexpr int V_TILE = HEAD_DIM * BKS * 2;       // [128][128] bf16 = 32 KB
constexpr int STAGE = K_TILE + V_TILE;
constexpr float kSumMax = 256.f;   // lazy-rescale bound on a lane's stage sum (2^8)

template <int NT>
__device__ __forceinline__ float tile_probs(const f32x16 (&st)[NT], bf16x8 (&pf)[NT][2],
                                            float m_ref, float sl2) {
  float ls = 0.f;
  const bf16x2 one = {(bf16)1.f, (bf16)1.f};
#pragma unroll
  for (int tt = 0; tt < NT; ++tt)
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      bf16x2 pr;
      pr[0] = (bf16)fast_exp2(fmaf(st[tt][i], sl2, -m_ref));
      pr[1] = (bf16)fast_exp2(fmaf(st[tt][i + 1], sl2, -m_ref));
      pf[tt][i >> 3][i & 7] = pr[0];
      pf[tt][i >> 3][(i & 7) + 1] = pr[1];
      ls = __builtin_amdgcn_fdot2_f32_bf16(pr, one, ls, false);
    }
  return ls;
}

// Partial results of the first and second half of the keys to one result: the
// weights of their outputs and the lse of both (log-sum-exp merge, -inf: no key).
__device__ __forceinline__ void half_weights(float la, float lb, float& wa, float& wb, float& lse) {
  const float m = fmaxf(la, lb);
  wa = wb = 0.f;
  lse = -INFINITY;
  if (m != -INFINITY) {
    wa = __expf(la - m);
    wb = __expf(lb - m);
    const float tot = wa + wb;
    lse = fmaf(__log2f(tot), 0.6931471805599453f, m);
    wa /= tot;
    wb /= tot;
  }
}
__device__ __forceinline__ float half_sum(float wa, float a, float wb, float b) {
  return fmaf(wb, b, wa * a);
}

// One query block of one head of one sequence against the key/value rows of
// its kv head.  Query row i (of Sq) may see key j (of Skv) iff j <= i + delta
// (causal) -- delta = 0 and Skv = Sq is plain causal self-attention; other
// offsets are one ring step of context-parallel attention -- and always
// j < Skv.  A row that sees no key gets O = 0 and lse = -inf, the neutral
// element of the log-sum-exp merge.  Q and O may be the same rows: a
// workgroup reads its queries before it writes, and no other one reads them.
// HV = 0: all keys.  HV = 1: the keys in two halves, by two workgroups, which
// leave their outputs in fp32 (half 0 in hv.p0, half 1 in hv.p1 and the row of O;
// lse in hv.l0 and lse) for half_merge_kernel.  HV = 2: the two halves one after
// the other, merged here by the same arithmetic.
template <bool CAUSAL, int KS, int HV>
__global__ __launch_bounds__(512, 1) void attn_fwd_kernel(
    HeadView Q, HeadView K, HeadView V, HeadView O, float* __restrict__ lse, int Sq, int Skv,
    int delta, int lse_heads, int nh, int h0, int G, int nqb, int nhb, FwdHalves hv) {
  constexpr int NQW = 8 / KS;            // waves along the query rows
  constexpr int NT = 4 / KS;             // 32-key tiles of a stage per wave
  constexpr int BQ = 32 * NQW;           // query rows per workgroup
  __shared__ __attribute__((aligned(1024))) char smem[2 * STAGE];
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wq = KS == 1 ? w : w % NQW, ks = KS == 1 ? 0 : w / NQW;
  const int r32 = lane & 31, g = lane >> 5;
  // Workgroup -> (query block, sequence, head), longest blocks first.
  const int half = HV == 1 ? blockIdx.x / (nqb * nhb) : 0;
  const int L = blockIdx.x - (HV == 1 ? half * nqb * nhb : 0);
  const int qb = nqb - 1 - L / nhb;
  const int u = (L % nhb) % nh;
  const int bi = (L % nhb) / nh;
  const int kvh = (h0 + u) / G;
  const int q0 = qb * BQ;
  const int qw = q0 + 32 * wq;              // first query row of this wave
  const int myq = qw + r32;                 // this lane's query row
  const bool row_ok = myq < Sq;

  // One head's K and V rows, 32-bit addressed; rows past Skv read as zero.
  const uint32_t rowb = (uint32_t)(K.row * 2);
  const uint32_t kv_bytes = (uint32_t)(Skv - 1) * rowb + 256u;
  const i32x4 rk = rsrc_words(K.p + bi * K.batch + kvh * K.head, kv_bytes);
  const i32x4 rv = rsrc_words(V.p + bi * V.batch + kvh * V.head, kv_bytes);
  uint32_t offk[4], offv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int blk = 4 * w + i;
    const int r = 4 * blk + (lane >> 4);       // stage row, 16 lanes per row
    offk[i] = r * rowb + ((uint32_t)((lane & 15) ^ (r & 15)) << 4);
    offv[i] = r * rowb + (((lane & 15) ^ tsw(r)) << 4);
  }

  // Stages of the workgroup (up to the last key its last row may see) and
  // the leading ones holding a key of this wave's part visible to it.
  const int max_st = (Skv + BKS - 1) / BKS;
  const int nst =
      CAUSAL ? max(0, min(max_st, (min(q0 + BQ, Sq) + delta + BKS - 1) / BKS)) : max_st;
  const int k_part = 32 * NT * ks;          // first key of this wave's part of a stage
  const int nw = qw >= Sq ? 0
                 : CAUSAL ? max(0, min(nst, (qw + 32 + delta - k_part + BKS - 1) / BKS))
                          : nst;
  // Last visible key of this lane's row and of the wave's first row.
  const int lim = CAUSAL ? min(myq + delta, Skv - 1) : Skv - 1;
  const int lim_w = CAUSAL ? min(qw + delta, Skv - 1) : Skv - 1;
  const uint32_t lds0 = lds_address(smem);
  // Stages j0 .. j1 - 1 of the walk.
  int j0 = 0, j1 = nst;
  if (HV == 1 && half > 0) j0 = min(hv.stage, nst);
  else if (HV > 0) j1 = min(hv.stage, nst);
  auto first_copies = [&]() {
    if (j0 < j1) {
      const uint32_t soff = HV == 0 ? 0 : (uint32_t)j0 * BKS * rowb;
      const uint32_t to = lds0 + (HV == 0 ? 0 : (j0 & 1) * STAGE);
      copy4_b128(rk, offk, soff, to + 4096 * w);
      copy4_b128(rv, offv, soff, to + K_TILE + 4096 * w);
    }
  };
  first_copies();

  // Q^T B-operand fragments for the whole key loop: lane = query column,
  // k-group g covers head-dim [16s + 8g, 16s + 8g + 8).
  bf16x8 qf[8];
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[s][e] = (bf16)0.f;
  if (row_ok) {
    const bf16* qp = Q.p + bi * Q.batch + u * Q.head + myq * Q.row + 8 * g;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
  }

  f32x16 oacc[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.f;
  // Reference max of the scaled scores (log2 domain): a finite stand-in for
  // -inf, so that a stage whose keys are all masked for a row leaves it at
  // p = 0 rather than producing 0 * inf.
  float m_ref = -1e30f;
  float l_run = 0.f;         // this lane's partial row sum
  f32x16 prev[HV == 2 ? 4 : 1];      // the first half's output and lse
  float prev_lse = 0.f;
  const float sl2 = 1.4426950408889634f * 0.08838834764831845f;  // log2(e)/sqrt(128)

  for (int walk = 0; walk < (HV == 2 ? 2 : 1); ++walk) {
    for (int j = j0; j < j1; ++j) {
      char* buf = smem + (j & 1) * STAGE;
      wait_vmem();
      __syncthreads();   // stage j landed for all waves; stage j-1's buffer is free
      const uint32_t nsoff = j + 1 < j1 ? (uint32_t)(j + 1) * BKS * rowb : 0;
      const uint32_t nlds = lds0 + ((j + 1) & 1) * STAGE;
      i32x4 nk = rk, nv = rv;
      if (j + 1 == j1) nk[2] = nv[2] = 0;
      if (j >= nw) {                          // whole stage masked for this wave
        copy4_b128(nk, offk, nsoff, nlds + 4096 * w);
        copy4_b128(nv, offv, nsoff, nlds + K_TILE + 4096 * w);
        continue;
      }
      {
        const int kb = j * BKS + k_part;
        f32x16 st[NT];
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
          for (int i = 0; i < 16; ++i) st[tt][i] = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
          for (int tt = 0; tt < NT; ++tt)
            st[tt] = mfma32x32x16(lds_read_b128(buf, swz256(k_part + 32 * tt + r32, 2 * s + g)),
                                  qf[s], st[tt]);
        // Keep six K fragment reads in flight ahead of the MFMAs: left alone,
        // the scheduler reads two, waits for them and multiplies, exposing the
        // LDS latency every two MFMAs.
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
        for (int i = 0; i < 8 * NT - 6; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
        // The next stage's copies follow the two blocks of products they can hide
        // behind: a wave stands still while the CU takes them, and at the top of
        // the stage nothing of it is under way.  Against there: one head over 4096
        // keys 43 -> 39 us, 8 heads over 4096 56 -> 52, 4 over 8192 90 -> 86, long
        // calls, where other waves fill the gap, within 0.5 %.
        copy4_b128(nk, offk, nsoff, nlds + 4096 * w);
        // Mask keys past the row's last visible key (wave-uniform test first).
        if (kb + 32 * NT - 1 > lim_w) {
#pragma unroll
          for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int key = kb + 32 * tt + 8 * (i >> 2) + 4 * g + (i & 3);
              if (key > lim) st[tt][i] = -INFINITY;
            }
        }
        bf16x8 pf[NT][2];
        float ls = tile_probs(st, pf, m_ref, sl2);
        if (__builtin_amdgcn_ballot_w64(!(ls <= kSumMax)) != 0) {
          float mx = st[0][0];
#pragma unroll
          for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, st[tt][i]);
          mx = fmaxf(mx, __shfl_xor(mx, 32)) * sl2;
          const float m_new = fmaxf(m_ref, mx);
          const float alpha = fast_exp2(m_ref - m_new);
          m_ref = m_new;
          l_run *= alpha;
#pragma unroll
          for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[dt][i] *= alpha;
          ls = tile_probs(st, pf, m_ref, sl2);
        }
        copy4_b128(nv, offv, nsoff, nlds + K_TILE + 4096 * w);
        l_run += ls;
#pragma unroll
        for (int c = 0; c < 2 * NT; ++c)
#pragma unroll
          for (int dt = 0; dt < 4; ++dt)
            oacc[dt] = mfma32x32x16(tr_operand(buf + K_TILE, k_part + 16 * c, 32 * dt, lane),
                                    pf[c >> 1][c & 1], oacc[dt]);
        // Stream the V^T fragments: four (eight transposing reads) ahead, then
        // two reads per MFMA (the default schedule issued bursts of eight
        // reads and waited between them).
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
        for (int i = 0; i < 8 * NT - 4; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
      }
    }

    wait_vmem();       // the last stage's empty copies (to LDS) have ended
    float l_tot = l_run + __shfl_xor(l_run, 32);
    if (KS > 1) {
      // Fold the KS parts of every row in fp32, in ascending key order: parts
      // 1.. pass (m_ref, l, acc) through the stage buffers (16 KB per wave).
      float* fold = reinterpret_cast<float*>(smem);
      float* fold_ml = fold + (KS - 1) * NQW * 4096;
      __syncthreads();   // every wave is done reading the last stage, and copying
      if (ks > 0) {
        const int slot = (ks - 1) * NQW + wq;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            f32x4 v;
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b] = oacc[dt][4 * a + b];
            *reinterpret_cast<f32x4*>(fold + slot * 4096 + (4 * dt + a) * 256 + lane * 4) = v;
          }
        fold_ml[slot * 128 + lane] = m_ref;
        fold_ml[slot * 128 + 64 + lane] = l_tot;
      }
      __syncthreads();
      if (HV < 2 && ks > 0) return;
#pragma unroll
      for (int p = 1; p < KS; ++p) {
        if (HV == 2 && ks > 0) break;
        const int slot = (p - 1) * NQW + wq;
        const float m_p = fold_ml[slot * 128 + lane], l_p = fold_ml[slot * 128 + 64 + lane];
        const float m_new = fmaxf(m_ref, m_p);
        const float a0 = fast_exp2(m_ref - m_new), a1 = fast_exp2(m_p - m_new);
        m_ref = m_new;
        l_tot = l_tot * a0 + l_p * a1;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            const f32x4 v =
                *reinterpret_cast<const f32x4*>(fold + slot * 4096 + (4 * dt + a) * 256 + lane * 4);
#pragma unroll
            for (int b = 0; b < 4; ++b) oacc[dt][4 * a + b] = oacc[dt][4 * a + b] * a0 + v[b] * a1;
          }
      }
    }
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;   // no visible key: O = 0
    const float row_lse =
        l_tot > 0.f ? (m_ref + __log2f(l_tot)) * 0.6931471805599453f : -INFINITY;
    if (HV == 2 && walk == 0) {
#pragma unroll
      for (int dt = 0; dt < (HV == 2 ? 4 : 0); ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          prev[dt][i] = oacc[dt][i] * inv;
          oacc[dt][i] = 0.f;
        }
      prev_lse = row_lse;
      m_ref = -1e30f;
      l_run = 0.f;
      j0 = j1;
      j1 = nst;
      __syncthreads();   // the folded parts have been read
      first_copies();
      continue;
    }
    if (!row_ok || ks > 0) return;
    bf16* op = O.p + bi * O.batch + u * O.head + myq * O.row;
    float* lp = lse + ((int64_t)bi * lse_heads + h0 + u) * Sq + myq;
    if (HV == 1) {
      const int64_t r = (int64_t)u * Sq + myq;
      float* lo = half > 0 ? hv.p1 + r * 64 : hv.p0 + r * HEAD_DIM;
      float* hi = half > 0 ? reinterpret_cast<float*>(op) : lo + 64;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          f32x4 ov;
#pragma unroll
          for (int b = 0; b < 4; ++b) ov[b] = oacc[dt][4 * a + b] * inv;
          *reinterpret_cast<f32x4*>((dt < 2 ? lo : hi) + 32 * (dt & 1) + 8 * a + 4 * g) = ov;
        }
      if (g == 0) *(half > 0 ? lp : hv.l0 + r) = row_lse;
      return;
    }
    float wa = 0.f, wb = 0.f, both = 0.f;
    if (HV == 2) half_weights(prev_lse, row_lse, wa, wb, both);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        bf16x4 ov;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          float x = oacc[dt][4 * a + b] * inv;
          if (HV == 2) x = half_sum(wa, prev[HV == 2 ? dt : 0][4 * a + b], wb, x);
          ov[b] = (bf16)x;
        }
        *reinterpret_cast<bf16x4*>(op + 32 * dt + 8 * a + 4 * g) = ov;
      }
    if (g == 0) *lp = HV == 2 ? both : row_lse;
  }
}

// The two halves' fp32 outputs of HV = 1 to o and lse: sixteen lanes a row (s, h)
// of o [Sq, H, d], 8 values each.  Half 1's upper 64 values lie in the row of o
// itself; all of a row's lanes are in one wave and read before any writes.
__global__ __launch_bounds__(256) void half_merge_kernel(FwdHalves hv, HeadView O,
                                                         float* __restrict__ lse, int Sq, int H) {
  const int64_t r = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);     // h * Sq + s
  if (r >= (int64_t)H * Sq) return;
  const int c = threadIdx.x & 15;
  bf16* op = O.p + (r / Sq) * O.head + (r % Sq) * O.row;
  const float* pa = hv.p0 + r * HEAD_DIM + 8 * c;
  const float* pb = (c < 8 ? hv.p1 + r * 64 : reinterpret_cast<const float*>(op) - 64) + 8 * c;
  const f32x4 a0 = *reinterpret_cast<const f32x4*>(pa), a1 = *reinterpret_cast<const f32x4*>(pa + 4);
  const f32x4 b0 = *reinterpret_cast<const f32x4*>(pb), b1 = *reinterpret_cast<const f32x4*>(pb + 4);
  float wa, wb, both;
  half_weights(hv.l0[r], lse[r], wa, wb, both);
  bf16x8 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    out[e] = (bf16)half_sum(wa, a0[e], wb, b0[e]);
    out[4 + e] = (bf16)half_sum(wa, a1[e], wb, b1[e]);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no store before the loads above
  *reinterpret_cast<bf16x8*>(op + 8 * c) = out;
  if (c == 0) lse[r] = both;
}

}  // namespace

// The waves of a workgroup cover 256, 128 or 64 query rows (1, 2 or 4 key
// parts).  More parts make more, shorter workgroups, each stage of which
// feeds less work per barrier and per byte copied: at a full chip 2 parts run
// at 0.87 and 4 parts at 0.72 of the rate of one (32768 x 32768 keys, 8 heads,
// all visible: 3515 / 4025 / 4809 us).  So the fewest parts whose
// workgroups still fill the 256 CUs, in 256-row blocks x heads (the
// chunk size and the batch do not enter, so they do not change a bit):
//   every key visible: one round of equal blocks.  128 blocks 508 / 651 us
//     (2 / 1 parts, 32768 rows, 1 head), 256 blocks 1009 / 883 (2 heads);
//     64 blocks 160 / 217 us (4 / 2 parts, 16384 rows, 1 head), 128 blocks
//     603 / 508 (32768 rows).
//   causal: the last block is twice the mean, and a single round is as long
//     as that.  256 blocks 269 / 354 us (2 / 1 parts, 16384 rows, 4 heads), 512
//     blocks 524 / 466 (8 heads); 128 blocks 171 / 223 us (4 / 2 parts, 16384
//     rows, 2 heads), 256 blocks 326 / 269.  Between the measured counts the
//     lines lie where the longest block of the coarser split takes as
//     long as all blocks of the finer one spread over the chip.
int attn_fwd_key_parts(int64_t Sq, int64_t Skv, int64_t delta, int Hq, int causal) {
  const int64_t blocks = (Sq + 255) / 256 * Hq;
  const bool all = !causal || delta >= Skv - 1;
  if (blocks > (all ? 128 : 448)) return 1;
  return blocks > (all ? 64 : 224) ? 2 : 4;
}

hipError_t launch_attn_fwd(const HeadView& Q, const HeadView& K, const HeadView& V,
                           const HeadView& O, float* lse, int64_t Sq, int64_t Skv, int64_t delta,
                           int64_t B, int lse_heads, int nh, int h0, int G, int causal, int parts,
                           hipStream_t st) {
  const int bq = 256 / parts;
  const int nqb = (int)((Sq + bq - 1) / bq);
  // Offsets beyond either length change nothing: clamp into int range.
  const int dl = (int)(delta < -Sq ? -Sq : delta > Skv ? Skv : delta);
  const int nhb = (int)(nh * B);
  dim3 grid((unsigned)(nqb * nhb));
#define UPIPE_FWD(C, P)                                                                       \
  hipLaunchKernelGGL((attn_fwd_kernel<C, P, 0>), grid, dim3(512), 0, st, Q, K, V, O, lse, (int)Sq, \
                     (int)Skv, dl, lse_heads, nh, h0, G, nqb, nhb, FwdHalves{})
  if (causal) {
    if (parts == 1) UPIPE_FWD(true, 1);
    else if (parts == 2) UPIPE_FWD(true, 2);
    else UPIPE_FWD(true, 4);
  } else {
    if (parts == 1) UPIPE_FWD(false, 1);
    else if (parts == 2) UPIPE_FWD(false, 2);
    else UPIPE_FWD(false, 4);
  }
#undef UPIPE_FWD
  return hipGetLastError();
}

// At most 128 queries are two workgroups a head, each a chain of 1.07 us for every
// stage of keys on a chip that is nearly idle; over two workgroups the chain is half
// as long.  One | two halves side by side, us: 128 queries of 4 heads on one
// key/value head, 16384 keys 144 | 77, 131072 1096 | 546; of 8 heads on 8, 131072
// 1715 | 861.  Where the workspace holds no outputs of halves (one key/value head,
// few heads a chunk) they run one after the other, 3 us longer than one piece:
// 8192 keys 68 | 71, 16384 144 | 145, 131072 1095 | 1083, so not below.  From 129
// queries on the workgroups share the keys they read in L2 and one piece is
// faster than the two halves by separate launches were (160 queries, 16384 keys 138).
int attn_fwd_half_stage(int64_t Sq, int64_t Skv, int64_t delta, int causal) {
  const int64_t seen = causal ? std::min(Skv, Sq + delta) : Skv;
  return Sq > 128 || seen <= 8192 ? 0 : (int)((seen + 2 * BKS - 1) / (2 * BKS));
}

FwdHalves attn_fwd_halves(int stage, int64_t Sq, int nh, char* room, size_t bytes) {
  const int64_t rows = Sq * nh;
  FwdHalves hv;
  hv.stage = stage;
  if (room != nullptr && bytes / ((HEAD_DIM + 64 + 1) * 4) >= (size_t)rows) {
    hv.p0 = (float*)room;
    hv.p1 = hv.p0 + rows * HEAD_DIM;
    hv.l0 = hv.p1 + rows * 64;
  }
  return hv;
}

hipError_t launch_attn_fwd_halves(const HeadView& Q, const HeadView& K, const HeadView& V,
                                  const HeadView& O, float* lse, int64_t Sq, int64_t Skv,
                                  int64_t delta, int lse_heads, int nh, int h0, int G, int causal,
                                  const FwdHalves& hv, hipStream_t st) {
  const int nqb = (int)((Sq + 63) / 64);
  const int dl = (int)(delta < -Sq ? -Sq : delta > Skv ? Skv : delta);
#define UPIPE_FWD(C, HV)                                                                        \
  hipLaunchKernelGGL((attn_fwd_kernel<C, 4, HV>), dim3((unsigned)(nqb * nh * (HV == 1 ? 2 : 1))), \
                     dim3(512), 0, st, Q, K, V, O, lse, (int)Sq, (int)Skv, dl, lse_heads, nh,   \
                     h0, G, nqb, nh, hv)
  if (causal) {
    if (hv.p0 != nullptr) UPIPE_FWD(true, 1);
    else UPIPE_FWD(true, 2);
  } else {
    if (hv.p0 != nullptr) UPIPE_FWD(false, 1);
    else UPIPE_FWD(false, 2);
  }
#undef UPIPE_FWD
  return hipGetLastError();
}

hipError_t launch_half_merge(const FwdHalves& hv, const HeadView& O, float* lse, int64_t Sq, int nh,
                             hipStream_t st) {
  hipLaunchKernelGGL(half_merge_kernel, dim3((unsigned)((Sq * nh + 15) / 16)), dim3(256), 0, st, hv,
                     O, lse, (int)Sq, nh);
  return hipGetLastError();
}

}  // namespace upipe
