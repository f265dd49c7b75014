// Causal GQA flash-attention backward for gfx950.
//
// Analytic gradient of softmax attention (paper Section 2.1), with the
// probabilities rebuilt from the saved row log-sum-exp (staged as -sqrt(d) lse,
// the initial value of each row's score accumulator):
//   P_ij  = exp(q_i.k_j/sqrt d - lse_i),   D_i = dO_i . O_i
//   dS_ij = P_ij (dO_i . v_j - D_i)
//   dV_j += sum_i P_ij dO_i,   dK_j += sum_i dS_ij q_i / sqrt d,
//   dQ_i  = sum_j dS_ij k_j / sqrt d.
// Two kernels, no atomics, one fixed summation order:
//   dkdv: a workgroup owns 128 keys of one key/value head (4 waves x 32 keys,
//         K and V fragments in registers; or 64 keys, two waves to each 32) and
//         walks the group's query heads in ascending order and, within a head,
//         the 128-row query tiles from the last one down to its diagonal
//         (each tile as 64-row halves, upper first, and each half as two
//         32-row subtiles, upper first), so that all resident workgroups
//         read the same query tiles at about the same time (shared L2 lines).
//         Long sequences: its fp32 dK/dV accumulators start from the values
//         the previous launch left in the workspace (UPipe keeps per-group
//         dK/dV accumulators alive across stages, Appendix A), so any chunk
//         size U gives bit-identical sums.  Shorter ones: the walk is cut
//         into segments side by side, whose sums are added in their order.
//   dq:   a workgroup owns 256 query rows of one head (8 waves) and walks
//         64-key stages in ascending order, recomputing P and dS; or 128 or 64
//         rows, with the keys of a 128-key stage split over the waves.
// What bounds them: at full chip, MFMA issue (dK/dV) and the power limit (dQ);
// short of 512 key blocks or 256-row blocks, the chip's filling.  Against one
// launch per chunk on packed copies, whole backward, one key/value head:
// 8192 rows of 4 heads (U = 1) 1882 -> 304 us, 32768 of 8 (U = 2) 11.1 -> 6.7 ms.
// Tiles reach LDS through buffer->LDS copies issued one tile ahead.
// Transposed operands are read out of row-major tiles (common.h, tr_operand).
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace upipe {

namespace {

constexpr float kSl2 = 1.4426950408889634f * 0.08838834764831845f;  // log2(e)/sqrt(128)
constexpr float kScale = 0.08838834764831845f;                      // 1/sqrt(128)

// ------------------------------------------------------------------ dK / dV
// LDS stage for one tile of QT query rows of one head: Q and dO rows
// [QT][128] (256-B rows, transposing-read swizzle), then lse and D [QT].  The
// B operands of dV += P^T dO and dK += dS^T Q are read out of the rows with
// transposing LDS reads, so no [d][S] copies of Q and dO are needed.  A tile
// is consumed as pairs of 32-row subtiles, the upper 64 rows first.
constexpr int QT = 128;
constexpr int ROWT = QT * HEAD_DIM * 2;
constexpr int OFF_Q = 0, OFF_DO = ROWT, OFF_LSE = 2 * ROWT, OFF_D = OFF_LSE + QT * 4;
constexpr int KV_STAGE = 2 * ROWT + QT * 8;
constexpr int KV_BLK = ROWT / 1024 / 4;     // 1 KB blocks per wave per array

struct QStageSrc {
  i32x4 q, dO, lse, D;
  uint32_t rowb;              // bytes from one row of Q or dO to the next
};

// The copies of one tile by one wave: KV_BLK blocks of 1 KB each of Q and dO rows,
// the QT lse values by wave 0 and the QT D values by wave 1 (16 bytes a lane).
// A CU takes about 20 clocks per 1 KB copy, and a wave that issues more than it
// takes stands still, products and all: issued together at the top of a tile,
// the copies of the next one held every wave for 1320 of the tile's 8100 clocks.
// So they go out in pair_step, in its two regions that are all products.  Against
// the top of the tile that is, for dK/dV of 4 heads over 1, 7 % at S = 8192 (202 ->
// 188 us), 4 % at 32768, 3 to 6 % at 65536.  Spread over all four regions, or all in
// one, they gain about half of it.
struct TileCopy {
  QStageSrc r;
  uint32_t row0;    // first query row of the tile
  uint32_t lds;     // LDS address of the stage
  int w;
  uint32_t vb;      // this lane's 16 bytes in the wave's first block: a row (16 lanes each),
                    // its chunk swizzled for the transposing reads

  // Blocks i0 .. i0 + n - 1 of this wave's (both even).
  __device__ __forceinline__ void blocks(int i0, int n) const {
#pragma unroll
    for (int i = i0; i < i0 + n; i += 2) {
      const uint32_t off = (vb ^ ((i & 3) << 4)) + 4 * i * r.rowb;
      const uint32_t off1 = (vb ^ (((i + 1) & 3) << 4)) + 4 * (i + 1) * r.rowb;
      copy2x2_b128<OFF_DO - OFF_Q>(r.q, r.dO, off, off1, row0 * r.rowb,
                                   lds + OFF_Q + (KV_BLK * w + i) * 1024);
    }
  }
  __device__ __forceinline__ void rows(int lane) const {
    if (lane < QT / 4) {
      if (w == 0) copy_b128(r.lse, lane * 16u, row0 * 4u, lds + OFF_LSE);
      else if (w == 1) copy_b128(r.D, lane * 16u, row0 * 4u, lds + OFF_D);
    }
  }
};

// Operand fragments of one block of 16 MFMAs.
struct Frags {
  bf16x8 f[16];
};

// S^T / dP^T block of one 32-row subtile (rows `sub`..+31 of the tile):
// fragment 2 s + 0 is Q, 2 s + 1 is dO, both for head-dim 16 s..
__device__ __forceinline__ void read_sdp(const char* buf, int sub, int r32, int g, Frags& fr) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    fr.f[2 * s] = lds_read_b128(buf + OFF_Q, swzt(sub + r32, 2 * s + g));
    fr.f[2 * s + 1] = lds_read_b128(buf + OFF_DO, swzt(sub + r32, 2 * s + g));
  }
}

// dV / dK block of one subtile: fragment 4 dt + 2 kt + 0 is dO, + 1 is Q, as
// B operands with head-dim columns 32 dt.. and the 16 query rows sub + 16 kt..
__device__ __forceinline__ void read_dvdk(const char* buf, int sub, int lane, Frags& fr) {
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      fr.f[4 * dt + 2 * kt] = tr_operand(buf + OFF_DO, sub + 16 * kt, 32 * dt, lane);
      fr.f[4 * dt + 2 * kt + 1] = tr_operand(buf + OFF_Q, sub + 16 * kt, 32 * dt, lane);
    }
}

// Accumulator seeds of the 32-row subtile at rows `sub`.. of the tile, in the
// MFMA C layout (element 4a + b is row sub + 8a + 4g + b), loaded from the
// staged rows straight into the accumulators: the score accumulator starts at
// -sqrt(d) lse of its row, so that it ends at q.k - sqrt(d) lse and
// P = exp2(acc log2(e) / sqrt(d)) needs no lse term; the dP accumulator
// starts at D, and the value fragments come negated, so that chain ends at
// D - dP and dS needs no subtraction: P (D - dP) = -dS.  A pair's seeds are
// read before its fragments: LDS reads complete in order, and a seed read
// behind a burst of fragment reads would wait for the whole burst.
__device__ __forceinline__ void subtile_seed(const char* buf, int sub, int g, f32x16& sacc,
                                             f32x16& pacc) {
  const float* Dl = reinterpret_cast<const float*>(buf + OFF_D) + sub;
  const float* Ll = reinterpret_cast<const float*>(buf + OFF_LSE) + sub;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const f32x4 d4 = *reinterpret_cast<const f32x4*>(Dl + 8 * a + 4 * g);
    const f32x4 l4 = *reinterpret_cast<const f32x4*>(Ll + 8 * a + 4 * g);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      pacc[4 * a + b] = d4[b];
      sacc[4 * a + b] = l4[b];
    }
  }
}

// S^T and D - dP^T of one subtile from its fragments (16 MFMAs), on top of
// the seeds.
__device__ __forceinline__ void subtile_sdp(const Frags& fr, const bf16x8 (&kf)[8],
                                            const bf16x8 (&nvf)[8], f32x16& sacc, f32x16& pacc) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    sacc = mfma32x32x16(fr.f[2 * s], kf[s], sacc);
    pacc = mfma32x32x16(fr.f[2 * s + 1], nvf[s], pacc);
  }
}

// P and -dS of one subtile as bf16 A operands, from its lse-seeded scores
// and D - dP.  Negation is exact and commutes with rounding, so the dK
// accumulators carry exactly -dK (the final scale is -1/sqrt d).  No masking
// here (subtile_mask).
__device__ __forceinline__ void subtile_pds(const f32x16& sacc, const f32x16& pacc,
                                            bf16x8 (&pf)[2], bf16x8 (&sf)[2]) {
  float p[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) p[i] = fast_exp2(sacc[i] * kSl2);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    pf[i >> 3][i & 7] = (bf16)p[i];
    sf[i >> 3][i & 7] = (bf16)(p[i] * pacc[i]);
  }
}

// Subtiles across the diagonal (wave-uniform `diag`; first row qs): zero the
// P and dS entries of keys after the row, by selection (unmasked they may be
// inf or NaN).  This runs after the conversions and between two regions: a
// branch ends the compiler's scheduling block, and inside a region it would
// split the MFMA / VALU interleave in two.
template <bool CAUSAL>
__device__ __forceinline__ void subtile_mask(uint32_t qs, uint32_t mykey, bool diag, int g,
                                             bf16x8 (&pf)[2], bf16x8 (&sf)[2]) {
  if (CAUSAL && diag) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (mykey > qs + 8 * (i >> 2) + 4 * g + (i & 3)) {
        pf[i >> 3][i & 7] = (bf16)0.f;
        sf[i >> 3][i & 7] = (bf16)0.f;
      }
  }
}

__device__ __forceinline__ void dvdk_products(const Frags& fr, const bf16x8 (&pf)[2],
                                              const bf16x8 (&sf)[2], f32x16 (&dva)[4],
                                              f32x16 (&dka)[4]) {
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      dva[dt] = mfma32x32x16(pf[kt], fr.f[4 * dt + 2 * kt], dva[dt]);
      dka[dt] = mfma32x32x16(sf[kt], fr.f[4 * dt + 2 * kt + 1], dka[dt]);
    }
}

// Scheduling request for a region of 16 MFMAs and the VALU work of one
// subtile's P and dS: one MFMA after every few VALU instructions, so the
// matrix unit and the vector ALU of the one wave on the SIMD work side by
// side (the region's LDS reads are left to the scheduler: asking for them
// first bunched the first MFMAs behind them).
constexpr int KV_NV = 5;   // VALU instructions requested between two MFMAs
// Region A (no VALU): its 16 MFMAs with the 32 transposing reads of the
// next block's fragments, two per MFMA; region D with the next pair's
// fragment reads, one per MFMA.
template <int NDS>
__device__ __forceinline__ void interleave_mfma_lds() {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, NDS, 0);
  }
}
__device__ __forceinline__ void interleave_mfma_valu() {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, KV_NV, 0);
  }
}

// One pair of subtiles (rows base..base+63 of the tile), in four fenced
// regions so that each block of 16 MFMAs shares its region with VALU work it
// does not depend on:
//   A: S/dP products of the upper subtile
//   B: S/dP products of the lower subtile   | P, dS of the upper subtile
//   C: dV/dK products of the upper subtile  | P, dS of the lower subtile
//   D: dV/dK products of the lower subtile
// The LDS fragments of each block are read one region ahead; fa holds the
// upper subtile's S / dP fragments on entry, and with PF it is refilled
// during region D (which has no other LDS reads) with those of the next
// pair of the tile.  Regions A and D each begin with 2 NB blocks of the next
// tile's copies, from `blk` on.  The lower subtile is computed even where only
// the upper one is needed: the diagonal mask then zeroes all of its P and dS.
// So is a pair that this wave's keys do not see at all; its dV / dK products then
// read the tile's upper pair (`dbuf` for `buf`), which the wave computes anyway:
// what a zero P or dS does to those rows is done already, where a row of the
// masked pair that holds an infinity or NaN would give 0 x NaN.
template <bool CAUSAL, bool PF, int NB>
__device__ __forceinline__ void pair_step(const TileCopy& next, int blk, const char* buf,
                                          const char* dbuf, int base, uint32_t qb, uint32_t kw,
                                          uint32_t mykey,
                                          int r32, int g, int lane, const bf16x8 (&kf)[8],
                                          const bf16x8 (&vf)[8],
                                          f32x16 (&dva)[4], f32x16 (&dka)[4], Frags& fa) {
  Frags fb;
  f32x16 s1, p1, s0, p0;
  bf16x8 pf1[2], sf1[2], pf0[2], sf0[2];
  const uint32_t q1 = qb + base + 32, q0 = qb + base;
  subtile_seed(buf, base + 32, g, s1, p1);
  subtile_seed(buf, base, g, s0, p0);
  __builtin_amdgcn_sched_barrier(0);
  read_sdp(buf, base, r32, g, fb);
  __builtin_amdgcn_sched_barrier(0);
  next.blocks(blk, 2 * NB);
  subtile_sdp(fa, kf, vf, s1, p1);                                            // A
  read_dvdk(dbuf, base + 32, lane, fa);
  interleave_mfma_lds<2>();
  __builtin_amdgcn_sched_barrier(0);
  subtile_sdp(fb, kf, vf, s0, p0);                                            // B
  subtile_pds(s1, p1, pf1, sf1);
  interleave_mfma_valu();
  __builtin_amdgcn_sched_barrier(0);
  subtile_mask<CAUSAL>(q1, mykey, q1 < kw + 31, g, pf1, sf1);
  dvdk_products(fa, pf1, sf1, dva, dka);                                      // C
  read_dvdk(dbuf, base, lane, fb);
  subtile_pds(s0, p0, pf0, sf0);
  interleave_mfma_valu();
  __builtin_amdgcn_sched_barrier(0);
  subtile_mask<CAUSAL>(q0, mykey, q0 < kw + 31, g, pf0, sf0);
  next.blocks(blk + 2 * NB, 2 * NB);
  dvdk_products(fb, pf0, sf0, dva, dka);                                      // D
  if (PF) {   // the next pair's upper subtile
    read_sdp(buf, base - 32, r32, g, fa);
    interleave_mfma_lds<1>();
  }
}

// Segments.  The lists of all key blocks are prefixes of one list, the query
// tiles from the last one down and within a tile the group's heads (beginning
// at the key block's own); it is cut at every T-th entry, so that the
// workgroups of one segment walk the same tiles side by side.  A key block (of
// 128 / QS keys) has whole segments and a last one of any length up to T.

// Key blocks whose list is longer than s segments: the first ones.
template <bool CAUSAL, int QS>
__host__ __device__ inline int seg_blocks(int s, int T, int G, int nqt) {
  if (!CAUSAL) return G * nqt > s * T ? QS * nqt : 0;
  const int tiles = nqt - s * (T / G);    // T is a multiple of G
  return tiles > 0 ? QS * tiles : 0;
}

// The x-th key block by the length of its last segment, longest first.  Tile j
// from the end has a list of G (j + 1) entries, the last segment of which is
// G (j % m + 1) long, m = T / G.
template <bool CAUSAL, int QS>
__device__ inline int by_last_segment(int x, int T, int G, int nqt) {
  if (!CAUSAL) return x;
  const int m = T / G, nt = nqt / m, rem = nqt % m, jx = x / QS;
  const int a = (m - rem) * nt;     // the lengths that only whole runs of m have
  int j;
  if (jx < a) j = (jx % nt) * m + m - 1 - jx / nt;
  else j = ((jx - a) % (nt + 1)) * m + rem - 1 - (jx - a) / (nt + 1);
  return QS * (nqt - 1 - j) + x % QS;
}

// QS = 1: a workgroup owns 128 keys, every wave takes all rows of a tile.
// QS = 2: 64 keys, two waves per 32 of them, one for each 64-row half of a tile;
// their sums are added through LDS.
// T = 0: one workgroup walks the whole list of its key block, head by head, on
// top of the carries.  T > 0: a workgroup per segment; where a key block has
// several, each leaves its fp32 sums in a slot and dkdv_fold_kernel adds them
// in list order.  Whole segments are dispatched first, then the last ones by
// length.
template <bool CAUSAL, int QS>
__global__ __launch_bounds__(256, 1) void attn_bwd_dkdv_kernel(
    HeadView Q, HeadView dO, const float* __restrict__ lse_c, const float* __restrict__ Dc,
    HeadView K, HeadView V, float* __restrict__ dK32, float* __restrict__ dV32, HeadView dk,
    HeadView dv, DkdvSlots slots, int64_t S, int64_t Sp, int U, int h0, int G) {
  constexpr int KB = 128 / QS;           // keys per workgroup
  __shared__ __attribute__((aligned(1024))) char smem[2 * KV_STAGE];
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wk = QS == 1 ? w : w & 1, qs = QS == 1 ? 0 : w >> 1;
  const int r32 = lane & 31, g = lane >> 5;
  const int T = slots.T;
  const uint32_t Spv = (uint32_t)Sp;
  const int nqt = (int)(Spv / QT);
  // Key/value head, key block and, with segments, segment and slot.
  int kv = blockIdx.y, kb = blockIdx.x, seg = 0, slot = 0;
  if (T > 0) {
    const int d = blockIdx.x, nw = slots.kv_heads * slots.whole;
    if (d < nw) {
      int i = d, base = 0, c;
      for (; i >= (c = seg_blocks<CAUSAL, QS>(seg + 1, T, G, nqt)) * slots.kv_heads; ++seg) {
        i -= c * slots.kv_heads;
        base += c;
      }
      kv = i / c;
      kb = i % c;
      slot = base + kb;
    } else {
      kv = (d - nw) % slots.kv_heads;
      kb = by_last_segment<CAUSAL, QS>((d - nw) / slots.kv_heads, T, G, nqt);
      seg = -1;
      slot = slots.whole + kb;
    }
  }
  const int kvh = h0 / G + kv;
  const int hlo = max(h0, kvh * G), hhi = min(h0 + U, (kvh + 1) * G);
  const uint32_t kb0 = kb * (uint32_t)KB;
  const uint32_t kw = kb0 + 32 * wk;     // first key of this wave
  const uint32_t mykey = kw + r32;       // key column owned by this lane
  const bool first = kvh * G >= h0;           // no earlier chunk touched kvh
  const bool last = (kvh + 1) * G <= h0 + U;  // no later chunk will
  const int qt_lo = CAUSAL ? (int)(kb0 / QT) : 0;   // lowest query tile needed
  const int per_head = nqt - qt_lo;
  int total = per_head * (hhi - hlo);
  int hh = hlo, qt = nqt - 1;     // head and query tile of the current iteration
  int left = 0;                   // heads of that tile yet to come (segments)
  bool whole = true;              // one workgroup has the whole list
  if (T > 0) {
    const int n = (total + T - 1) / T;
    whole = n == 1;
    if (seg < 0) {
      seg = n - 1;
      total -= seg * T;
    } else {
      total = T;
    }
    left = G - 1 - seg * T % G;
    hh += (seg * T + kb) % G;   // the heads share out the L2 channels of token-major rows
    qt -= seg * T / G;
  }

  auto srcs = [&](int hh) {
    QStageSrc r;
    const int64_t u = hh - h0;
    r.rowb = (uint32_t)(Q.row * 2);
    r.q = rsrc_words(Q.p + u * Q.head, (uint32_t)(S - 1) * r.rowb + 256u);
    r.dO = rsrc_words(dO.p + u * dO.head, (uint32_t)(S - 1) * r.rowb + 256u);
    r.lse = rsrc_words(lse_c + u * Sp, Spv * 4u);
    r.D = rsrc_words(Dc + u * Sp, Spv * 4u);
    return r;
  };

  const uint32_t lds0 = lds_address(smem);
  TileCopy next{srcs(hh), (uint32_t)(qt * QT), lds0, w, 0};
  next.vb = (4 * KV_BLK * w + (lane >> 4)) * next.r.rowb + (((lane & 15) ^ ((lane >> 4) << 2)) << 4);
  next.rows(lane);
  next.blocks(0, KV_BLK);

  // K and -V B-operand fragments (lane = key column, k = head dim); -V makes
  // the dP products count down from D.  Keys past S repeat the last one; their
  // sums are not used.
  bf16x8 kf[8], vf[8];
  {
    const uint32_t key = min(mykey, (uint32_t)S - 1);
    const bf16* kp = K.p + kvh * K.head + key * K.row + 8 * g;
    const bf16* vp = V.p + kvh * V.head + key * V.row + 8 * g;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      kf[s] = *reinterpret_cast<const bf16x8*>(kp + 16 * s);
      vf[s] = -*reinterpret_cast<const bf16x8*>(vp + 16 * s);
    }
    // They are only ever MFMA operands, which may come from AGPRs: placing
    // them there leaves the VGPRs to the score accumulators and the P / dS
    // arithmetic (fewer AGPR -> VGPR moves, no spills).
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      asm volatile("" : "+a"(kf[s]));
      asm volatile("" : "+a"(vf[s]));
    }
  }

  // Accumulators: C layout with lane = head-dim column 32*dt + r32 and
  // element i = key row kw + 8*(i/4) + 4*g + (i%4).
  f32x16 dka[4], dva[4];
  float* dK32h = dK32 + (int64_t)kvh * Sp * HEAD_DIM;
  float* dV32h = dV32 + (int64_t)kvh * Sp * HEAD_DIM;
  if (QS > 1 || first) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        dka[dt][i] = 0.f;
        dva[dt][i] = 0.f;
      }
  } else {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t off = (kw + 8 * (i >> 2) + 4 * g + (i & 3)) * HEAD_DIM + 32 * dt + r32;
        dka[dt][i] = dK32h[off];
        dva[dt][i] = dV32h[off];
      }
  }

  for (int it = 0; it < total; ++it) {
    char* buf = smem + (it & 1) * KV_STAGE;
    const uint32_t qb = qt * QT;
    // next tile: descending query tiles, then the next head; with segments
    // the next head round, then descending
    int nq = qt - 1, nh = hh;
    if (T > 0) {
      nh = hh + 1 < hhi ? hh + 1 : hlo;
      if (left-- > 0) nq = qt;
      else left = G - 1;
    } else if (qt == qt_lo) {
      nq = nqt - 1;
      nh = hh + 1;
    }
    wait_vmem();
    __syncthreads();   // this tile landed for all waves; the other buffer is free
    // After the last tile the copies read nothing (a source of no bytes, from
    // offset 0 on, gives zeros), so that no region has to ask.
    if (nh != hh) next.r = srcs(nh);
    if (it + 1 == total)
      next.r.q[2] = next.r.dO[2] = next.r.lse[2] = next.r.D[2] = 0;
    next.row0 = it + 1 < total ? nq * QT : 0;
    next.lds = lds0 + ((it + 1) & 1) * KV_STAGE;
    next.rows(lane);
    // Pairs of 32-row subtiles, upper rows first; the upper pair reads the lower
    // pair's first fragments in its region D.  A pair above the diagonal (only a
    // lower one can be) is computed too, and masked whole: the waves it concerns
    // would wait for the others, and a branch round it costs the kernel its
    // registers.
    const char* lower = buf + (CAUSAL && qb + 63 < kw ? 64 * HEAD_DIM * 2 : 0);
    Frags fa;
    if (QS == 1) {
      read_sdp(buf, 96, r32, g, fa);
      pair_step<CAUSAL, true, 1>(next, 0, buf, buf, 64, qb, kw, mykey, r32, g, lane, kf, vf, dva,
                                 dka, fa);
      pair_step<CAUSAL, false, 1>(next, 4, buf, lower, 0, qb, kw, mykey, r32, g, lane, kf,
                                  vf, dva, dka, fa);
    } else {
      const int base = 64 * qs;
      read_sdp(buf, base + 32, r32, g, fa);
      pair_step<CAUSAL, false, 2>(next, 0, buf, qs == 0 ? lower : buf, base, qb, kw, mykey, r32, g,
                                  lane, kf, vf, dva, dka, fa);
    }
    qt = nq;
    hh = nh;
  }

  wait_vmem();      // the last tile's empty copies (to LDS) have ended
  if (QS > 1) {   // rows 64.. of the tiles onto rows 0..63, in fp32
    float* fold = reinterpret_cast<float*>(smem) + wk * 8192 + lane * 4;
    __syncthreads();   // every wave is done reading the last tile, and copying
    if (qs > 0) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          f32x4 x, y;
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            x[b] = dka[dt][4 * a + b];
            y[b] = dva[dt][4 * a + b];
          }
          *reinterpret_cast<f32x4*>(fold + (4 * dt + a) * 256) = x;
          *reinterpret_cast<f32x4*>(fold + (16 + 4 * dt + a) * 256) = y;
        }
    }
    __syncthreads();
    if (qs > 0) return;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(fold + (4 * dt + a) * 256);
        const f32x4 y = *reinterpret_cast<const f32x4*>(fold + (16 + 4 * dt + a) * 256);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          dka[dt][4 * a + b] += x[b];
          dva[dt][4 * a + b] += y[b];
        }
      }
  }
  if (!whole || (QS == 1 && !last)) {
    // Slots [2][KB][128], carries [Sp][128]: the key's row of 128 floats.
    float* pk = dK32h + (int64_t)kw * HEAD_DIM;
    float* pv = dV32h + (int64_t)kw * HEAD_DIM;
    if (!whole) {
      pk = slots.at((int64_t)kv * slots.per_head + slot, 2 * KB * HEAD_DIM) +
           32 * wk * HEAD_DIM;
      pv = pk + KB * HEAD_DIM;
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t off = (8 * (i >> 2) + 4 * g + (i & 3)) * HEAD_DIM + 32 * dt + r32;
        pk[off] = dka[dt][i];
        pv[off] = dva[dt][i];
      }
  } else {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t key = kw + 8 * (i >> 2) + 4 * g + (i & 3);
        if (key < (uint64_t)S) {
          const int64_t e = 32 * dt + r32;
          dk.p[kvh * dk.head + key * dk.row + e] = (bf16)(dka[dt][i] * -kScale);
          dv.p[kvh * dv.head + key * dv.row + e] = (bf16)dva[dt][i];
        }
      }
  }
}

// The segments' sums of the key blocks that have several, added in list order:
// blockIdx.x = key block, y = key/value head; a thread has eight consecutive
// elements of one key's dK or dV.  Reads each slot once.
template <bool CAUSAL, int QS>
__global__ __launch_bounds__(256) void dkdv_fold_kernel(DkdvSlots slots, HeadView dk, HeadView dv,
                                                        int64_t S, int64_t Sp, int G) {
  constexpr int KB = 128 / QS;
  const int nqt = (int)(Sp / QT), kb = blockIdx.x / (KB / 8);
  const int kvh = blockIdx.y;
  const int e8 = ((blockIdx.x % (KB / 8)) * 256 + threadIdx.x) * 8;   // in [2][KB][128]
  const int64_t base = (int64_t)kvh * slots.per_head + kb;
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
  auto add = [&](int64_t i) {
    const float* p = slots.at(base + i, 2 * KB * HEAD_DIM) + e8;
    lo += *reinterpret_cast<const f32x4*>(p);
    hi += *reinterpret_cast<const f32x4*>(p + 4);
  };
  int64_t at = 0;
  int c;
  for (int s = 1; kb < (c = seg_blocks<CAUSAL, QS>(s, slots.T, G, nqt)); ++s) {
    add(at);
    at += c;
  }
  add(slots.whole);
  const bool is_v = e8 >= KB * HEAD_DIM;
  const int key = (e8 / HEAD_DIM) % KB + kb * KB, e = e8 % HEAD_DIM;
  if (key >= S) return;
  const float f = is_v ? 1.f : -kScale;
  bf16x8 out;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[i] = (bf16)(lo[i] * f);
    out[4 + i] = (bf16)(hi[i] * f);
  }
  const HeadView& d = is_v ? dv : dk;
  *reinterpret_cast<bf16x8*>(d.p + kvh * d.head + key * d.row + e) = out;
}

// ---------------------------------------------------------------------- dQ
// Workgroup = 8 waves of 32 query rows x a part of every stage's keys: 256 rows
// x 64-key stages, or, with the keys of 128-key stages split in 2 or 4 parts
// (attn_bwd_dq_key_parts), 128 or 64 rows, whose sums are added in fp32 through
// LDS.  LDS stage for one tile of keys: K and V rows (256-B rows).  The A
// operand of dQ^T = K^T . dS^T is read out of the K rows with transposing LDS
// reads, so no [d][S] copy of K is needed.
template <int KS>
struct DqTile {
  static constexpr int NQW = 8 / KS;                // waves along the query rows
  static constexpr int BQ = 32 * NQW;               // query rows per workgroup
  static constexpr int BK = KS == 1 ? 64 : 128;     // keys per stage
  static constexpr int NH = BK / 32 / KS;           // 32-key blocks of a stage per wave
  static constexpr int T = BK * HEAD_DIM * 2;
  static constexpr int OFF_K = 0, OFF_V = T;
  static constexpr int STAGE = 2 * T;
  static constexpr int BLK = T / 1024 / 8;          // 1 KB blocks per wave per tile
};
// K/V fragment reads kept in flight (backward, us, with 4 | 6 | 8: 4100 rows of 8 heads
// 177.6 | 179.3 | 179.7, 8192 of 4 309.2 | 311.5 | 309.8).
constexpr int DQ_LA = 4;

// Two of this wave's BLK 1 KB blocks (4 rows of 256 B each) of K rows and the
// same of V rows, i even, at byte offset `soff` of the head's rows; `lds` is the
// stage's LDS address.
template <int KS>
__device__ __forceinline__ void issue_kblocks(i32x4 rk, i32x4 rv,
                                              const uint32_t (&off)[DqTile<KS>::BLK], int i,
                                              uint32_t soff, uint32_t lds, int w) {
  using T = DqTile<KS>;
  copy2x2_b128<T::OFF_V - T::OFF_K>(rk, rv, off[i], off[i + 1], soff,
                                    lds + T::OFF_K + (T::BLK * w + i) * 1024);
}

// dQ may be the rows of Q or dO: a workgroup reads its rows before it writes
// them, and no other one reads them.
template <bool CAUSAL, bool ROPE, int KS>
__global__ __launch_bounds__(512, 1) void attn_bwd_dq_kernel(
    HeadView Q, HeadView dO, const float* __restrict__ lse_c, const float* __restrict__ Dc,
    HeadView K, HeadView V, HeadView dQ, int64_t S, int64_t Sp, int nh, int h0, int G, int nqb,
    int nhb, RopeArgs rope) {
  using T = DqTile<KS>;
  __shared__ __attribute__((aligned(1024))) char smem[2 * T::STAGE];
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wq = KS == 1 ? w : w % T::NQW, ks = KS == 1 ? 0 : w / T::NQW;
  const int r32 = lane & 31, g = lane >> 5;
  const int L = blockIdx.x;
  const int qb = nqb - 1 - L / nhb;
  const int row0 = L % nhb;                 // row of lse_c and D: sequence, head
  const int u = row0 % nh;
  const int bi = row0 / nh;
  const int kvh = (h0 + u) / G;
  const uint32_t Sv = (uint32_t)S;
  const uint32_t q0 = (uint32_t)qb * T::BQ;
  const uint32_t qw = q0 + 32 * wq;
  const uint32_t myq = qw + r32;
  const bool wave_ok = qw < Sv;
  const bool row_ok = myq < Sv;

  // One head's K and V rows, 32-bit addressed; rows past S read as zero.
  const uint32_t rowb = (uint32_t)(K.row * 2);
  const i32x4 rk = rsrc_words(K.p + bi * K.batch + kvh * K.head, (Sv - 1) * rowb + 256u);
  const i32x4 rv = rsrc_words(V.p + bi * V.batch + kvh * V.head, (Sv - 1) * rowb + 256u);
  const uint32_t lds0 = lds_address(smem);
  uint32_t off[T::BLK];
#pragma unroll
  for (int i = 0; i < T::BLK; ++i) {
    const int blk = T::BLK * w + i;
    const int r = 4 * blk + (lane >> 4);      // row of the tile, 16 lanes per row
    off[i] = r * rowb + (((lane & 15) ^ tsw(r)) << 4);
  }
  const int nst = (int)(((CAUSAL ? min(q0 + T::BQ, Sv) : Sv) + T::BK - 1) / T::BK);
#pragma unroll
  for (int i = 0; i < T::BLK; i += 2) issue_kblocks<KS>(rk, rv, off, i, 0, lds0, w);

  // Rows past S compute on the last row's values and are not written.
  bf16x8 qf[8], df[8];
  float nlse, Dq;   // nlse = -sqrt(d) lse: the score accumulator's seed
  {
    const uint32_t row = min(myq, Sv - 1);
    const bf16* qp = Q.p + bi * Q.batch + u * Q.head + row * Q.row + 8 * g;
    const bf16* dp = dO.p + bi * dO.batch + u * dO.head + row * dO.row + 8 * g;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      qf[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
      df[s] = *reinterpret_cast<const bf16x8*>(dp + 16 * s);
    }
    nlse = lse_c[row0 * Sp + row];
    Dq = Dc[row0 * Sp + row];
  }

  f32x16 qacc[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) qacc[dt][i] = 0.f;

  const int k_part = 32 * T::NH * ks;        // first key of this wave's part of a stage
  const uint32_t k_lane = T::OFF_K + k_part * 256 + swzt(r32, g);
  const uint32_t v_lane = T::OFF_V + k_part * 256 + swzt(r32, g);
  const uint32_t t_lane = T::OFF_K + k_part * 256 + tr_base(lane);
  // Stages with a key of this wave's part that a row of it may see come first.
  const int nw = !wave_ok ? 0
                 : CAUSAL ? min(nst, qw + 31 < (uint32_t)k_part ? 0 : (int)((qw + 31 - k_part) / T::BK) + 1)
                          : nst;
  int j = 0;
  for (; j < nw; ++j) {
    const uint32_t boff = (j & 1) * T::STAGE;
    wait_vmem();
    __syncthreads();   // tile j landed for all waves; tile j-1's buffer is free
    const uint32_t nsoff = j + 1 < nst ? (uint32_t)(j + 1) * T::BK * rowb : 0;
    const uint32_t nlds = lds0 + ((j + 1) & 1) * T::STAGE;
    i32x4 nk = rk, nv = rv;
    if (j + 1 == nst) nk[2] = nv[2] = 0;     // no next tile: zeros
    const uint32_t kb = (uint32_t)j * T::BK + k_part;
    const bool diag = CAUSAL ? (kb + 32 * T::NH - 1 > qw) : (kb + 32 * T::NH > Sv);
    // 32 keys at a time: one score and one dP accumulator live at a time,
    // which leaves registers for DQ_LA fragment reads in flight ahead of the
    // S / dP MFMAs (with two blocks' accumulators live the compiler kept one,
    // waiting before every MFMA).  The dQ products add a wave's 16-key steps
    // in ascending order.  The fragment addresses are exclusive-ors of three
    // bases: one register for each of them would spill.
    const uint32_t ka = k_lane + boff, va = v_lane + boff, ta = t_lane + boff;
#pragma unroll
    for (int hh = 0; hh < T::NH; ++hh) {
      f32x16 sacc, pacc;
#pragma unroll
      for (int i = 0; i < 16; ++i) { sacc[i] = nlse; pacc[i] = 0.f; }
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        sacc = mfma32x32x16(lds_read_b128(smem, (ka ^ (32 * s)) + 8192 * hh), qf[s], sacc);
        pacc = mfma32x32x16(lds_read_b128(smem, (va ^ (32 * s)) + 8192 * hh), df[s], pacc);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, DQ_LA, 0);
#pragma unroll
      for (int i = 0; i < 16 - DQ_LA; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, DQ_LA, 0);
      // The next tile's copies go out behind the products they can hide behind
      // (as in the forward).  Against the top of the tile, whole backward: 4100 rows
      // of 8 heads 182.7 -> 177.6 us, 2500 of 4 (every key visible) 127.9 -> 126.8, 8192
      // of 4 310.9 -> 309.2, 32768 of 4 3444 -> 3435.
      if (hh == 0) issue_kblocks<KS>(nk, nv, off, 0, nsoff, nlds, w);
      if (T::BLK > 2 && hh == T::NH - 1) issue_kblocks<KS>(nk, nv, off, 2, nsoff, nlds, w);
      bf16x8 sf[2];
      float p[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) p[i] = fast_exp2(sacc[i] * kSl2);
      if (diag) {   // wave-uniform
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const uint32_t key = kb + 32 * hh + 8 * (i >> 2) + 4 * g + (i & 3);
          const bool vis = CAUSAL ? (key <= myq) : (key < Sv);
          if (!vis) p[i] = 0.f;
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) sf[i >> 3][i & 7] = (bf16)(p[i] * (pacc[i] - Dq));
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
          qacc[dt] =
              mfma32x32x16(tr_operand_at(smem, ta, 32 * hh + 16 * c, dt), sf[c], qacc[dt]);
    }
  }

  // The others: only this wave's share of the copies.
  for (; j < nst; ++j) {
    wait_vmem();
    __syncthreads();
    if (j + 1 < nst)
#pragma unroll
      for (int i = 0; i < T::BLK; i += 2)
        issue_kblocks<KS>(rk, rv, off, i, (uint32_t)(j + 1) * T::BK * rowb,
                          lds0 + ((j + 1) & 1) * T::STAGE, w);
  }
  wait_vmem();       // the last stage's empty copies (to LDS) have ended
  if (KS > 1) {
    // Add the KS parts' sums in ascending key order: parts 1.. pass theirs
    // through the stage buffers (16 KB per wave).
    float* fold = reinterpret_cast<float*>(smem);
    __syncthreads();   // every wave is done reading the last stage
    if (ks > 0) {
      float* mine = fold + ((ks - 1) * T::NQW + wq) * 4096 + lane * 4;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          f32x4 v;
#pragma unroll
          for (int b = 0; b < 4; ++b) v[b] = qacc[dt][4 * a + b];
          *reinterpret_cast<f32x4*>(mine + (4 * dt + a) * 256) = v;
        }
    }
    __syncthreads();
    if (ks > 0) return;
#pragma unroll
    for (int p = 1; p < KS; ++p) {
      const float* part = fold + ((p - 1) * T::NQW + wq) * 4096 + lane * 4;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(part + (4 * dt + a) * 256);
#pragma unroll
          for (int b = 0; b < 4; ++b) qacc[dt][4 * a + b] += v[b];
        }
    }
  }
  if (!row_ok) return;
  if (ROPE) {   // dQ was taken with respect to rotated queries: turn it back
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int e = 32 * dt + 8 * (i >> 2) + 4 * g + (i & 3);
        float c, s;
        cos_sin_turns(rope_turn(rope.pos0 + myq, rope_turns_per_pos(e, rope.log2_base)), c, s);
        rope_pair(qacc[dt], qacc[dt + 2], i, c, s, true);
      }
  }
  bf16* op = dQ.p + bi * dQ.batch + u * dQ.head + myq * dQ.row + 4 * g;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      bf16x4 ov;
#pragma unroll
      for (int b = 0; b < 4; ++b) ov[b] = (bf16)(qacc[dt][4 * a + b] * kScale);
      *reinterpret_cast<bf16x4*>(op + 32 * dt + 8 * a) = ov;
    }
}

}  // namespace

hipError_t launch_attn_bwd_dkdv(const HeadView& Q, const HeadView& dO, const float* lse_c,
                                const float* D, const HeadView& K, const HeadView& V, float* dK32,
                                float* dV32, const HeadView& dk, const HeadView& dv, int64_t S,
                                int64_t Sp, int nh, int h0, int G, int causal, hipStream_t st) {
  if (Q.row != dO.row) return hipErrorInvalidValue;
  const int kv_lo = h0 / G, kv_hi = (h0 + nh - 1) / G;
  dim3 grid((unsigned)(Sp / 128), (unsigned)(kv_hi - kv_lo + 1));
#define UPIPE_DKDV(C)                                                                          \
  hipLaunchKernelGGL((attn_bwd_dkdv_kernel<C, 1>), grid, dim3(256), 0, st, Q, dO, lse_c, D, K, \
                     V, dK32, dV32, dk, dv, DkdvSlots{}, S, Sp, nh, h0, G)
  if (causal) UPIPE_DKDV(true);
  else UPIPE_DKDV(false);
#undef UPIPE_DKDV
  return hipGetLastError();
}

namespace {

int seg_blocks_of(int causal, int qs, int s, int T, int G, int nqt) {
  if (causal)
    return qs == 1 ? seg_blocks<true, 1>(s, T, G, nqt) : seg_blocks<true, 2>(s, T, G, nqt);
  return qs == 1 ? seg_blocks<false, 1>(s, T, G, nqt) : seg_blocks<false, 2>(s, T, G, nqt);
}

// Whole segments of one key/value head's lists that are not their last.
int64_t whole_segments(int causal, int qs, int T, int G, int nqt) {
  int64_t n = 0;
  for (int s = 1, c; (c = seg_blocks_of(causal, qs, s, T, G, nqt)) > 0; ++s) n += c;
  return n;
}

}  // namespace

// Chooses the keys of a workgroup (128 or 64) and the segment length T by the
// time they are expected to take, in units of one 128 x 128 tile on a full chip
// (about 4 us).  Measured, causal, d_model 4096 block, with the copies at the top of
// a tile, where the ratios below come from (T: workgroups, us):
//   8192 rows, 4 heads    T 20: 442, 207   32: 288, 214   40: 238, 182   64: 160, 258
//                         128: 96, 463     256: 64, 885 (no segments)
//   16384 rows, 4 heads   T 80: 476, 684   96: 408, 784   128: 320, 680  192: 240, 772
// A tile takes 3.25 us with few workgroups running, 4.1 with 256 (one per CU);
// with 64 keys 2.6 (causal; 0.72 of 128 keys' if every key is visible), for half
// the work but all of the copies, so 64 keys pay only where the slots that
// the workspace holds bound T and the launch is one round.  Whole segments run
// 256 at a time, then the last segments of the lists, of all lengths up to T,
// longest first: the shorter ones wait for a CU, and the next in order for
// that one's shader engine, so a second wave costs 0.3 T more than
// its longest.  A workgroup costs two tiles besides its list, the fold 1.5 and
// 0.016 per slot.
// Against a launch per head with one workgroup per key block (dK/dV with its fold):
// 512 rows, 2 heads 46 -> 23 us; 4096 rows, 8 heads on 2 935 -> 106; 8192 rows, 4 heads
// 895 -> 190; 32768 rows, 8 heads 7.0 -> 4.0 ms, 1028 tiles per CU at 3.9 us.
DkdvSplit dkdv_split(int64_t Sp, int Hkv, int G, int causal, size_t bytes0, size_t bytes1) {
  const int nqt = (int)(Sp / QT);
  DkdvSplit best;
  for (int qs = 1; qs <= 2; ++qs) {
    const size_t slot = (size_t)2 * (128 / qs) * HEAD_DIM * 4;
    const int64_t have = (int64_t)(bytes0 / slot + bytes1 / slot);
    // The longest list in n / 8 parts; equal lists in whole parts only.
    for (int n = 8; n <= 128; n += causal ? 1 : 8) {
      DkdvSplit p;
      p.qs = qs;
      p.T = causal ? G * ((8 * nqt + n - 1) / n) : (8 * G * nqt + n - 1) / n;
      p.whole = (int)whole_segments(causal, qs, p.T, G, nqt);
      const int64_t used = Hkv * (int64_t)(p.whole + seg_blocks_of(causal, qs, 1, p.T, G, nqt));
      if (used > have) continue;
      const int64_t blocks = (int64_t)Hkv * nqt * qs;
      const double busy = std::min(1.0, (blocks + Hkv * (double)p.whole) / 256);
      const double T = p.T * (qs == 1 ? 0.8 + 0.2 * busy : causal ? 0.64 : 0.58) + 2.0;
      const int64_t rest = causal ? blocks : 0;
      const int64_t whole = Hkv * (int64_t)p.whole + (causal ? 0 : blocks);
      if (qs > 1 && whole + rest > 288) continue;
      const int64_t rounds = whole / 256, extra = whole % 256, room = 256 - extra;
      double span = rounds * T;
      if (rest <= room) {
        if (rest + extra > 0) span += T;
      } else {
        // `room` of the others start at once, the rest (up to x long) as
        // those finish, the shortest first
        const double x = T * (rest - room) / rest;
        span += rest <= 2 * room ? std::max(T, 2 * x) + 0.3 * T
                                 : std::max(T, (extra + rest * 0.5) * T / 256 + 0.5 * T);
      }
      p.est = span + (used > 0 ? 1.5 + used * 0.016 / qs : 0);
      if (best.T == 0 || p.est < best.est) best = p;
    }
  }
  return best;
}

hipError_t launch_attn_bwd_dkdv_split(const HeadView& Q, const HeadView& dO, const float* lse_c,
                                      const float* D, const HeadView& K, const HeadView& V,
                                      const HeadView& dk, const HeadView& dv, int64_t S, int64_t Sp,
                                      int Hkv, int G, int causal, const DkdvSplit& p, char* region0,
                                      size_t bytes0, char* region1, hipStream_t st) {
  if (p.T < 1 || Q.row != dO.row) return hipErrorInvalidValue;
  const int nqt = (int)(Sp / QT);
  const size_t slot = (size_t)2 * (128 / p.qs) * HEAD_DIM * 4;
  DkdvSlots s;
  s.p0 = (float*)region0;
  s.p1 = (float*)region1;
  s.n0 = (int64_t)(bytes0 / slot);
  s.T = p.T;
  s.kv_heads = Hkv;
  s.whole = p.whole;
  const int c1 = seg_blocks_of(causal, p.qs, 1, p.T, G, nqt);   // blocks with several
  s.per_head = p.whole + c1;
  dim3 grid((unsigned)((nqt * p.qs + p.whole) * Hkv));
  dim3 fold((unsigned)(c1 * (128 / p.qs / 8)), (unsigned)Hkv);
#define UPIPE_DKDV(C, N)                                                                         \
  hipLaunchKernelGGL((attn_bwd_dkdv_kernel<C, N>), grid, dim3(256), 0, st, Q, dO, lse_c, D,      \
                     K, V, nullptr, nullptr, dk, dv, s, S, Sp, Hkv * G, 0, G);       \
  if (c1 > 0)                                                                                    \
  hipLaunchKernelGGL((dkdv_fold_kernel<C, N>), fold, dim3(256), 0, st, s, dk, dv, S, Sp, G)
  if (causal) {
    if (p.qs == 1) { UPIPE_DKDV(true, 1); }
    else { UPIPE_DKDV(true, 2); }
  } else {
    if (p.qs == 1) { UPIPE_DKDV(false, 1); }
    else { UPIPE_DKDV(false, 2); }
  }
#undef UPIPE_DKDV
  return hipGetLastError();
}

// As attn_fwd_key_parts, at the same lines: 512 blocks 700 / 756 us (1 / 2 parts,
// causal, 16384 rows, 8 heads), 256 blocks 511 / 381 (4 heads) and 430 with 4, 128
// blocks 288 / 221 (2 / 4 parts, 2 heads); every key visible 128 blocks 255 / 189
// (1 / 2 parts, 8192 rows, 4 heads), 256 blocks 344 / 368 (8 heads), 64 blocks 148 /
// 112 (2 / 4 parts, 2 heads).
int attn_bwd_dq_key_parts(int64_t S, int Hq, int causal) {
  const int64_t blocks = (S + 255) / 256 * Hq;
  if (blocks > (causal ? 448 : 128)) return 1;
  return blocks > (causal ? 224 : 64) ? 2 : 4;
}

hipError_t launch_attn_bwd_dq(const HeadView& Q, const HeadView& dO, const float* lse_c,
                              const float* D, const HeadView& K, const HeadView& V,
                              const HeadView& dQ, int64_t S, int64_t Sp, int64_t B, int nh, int h0,
                              int G, int causal, int parts, RopeArgs rope, hipStream_t st) {
  const int bq = 256 / parts;
  const int nqb = (int)((S + bq - 1) / bq);
  const int nhb = (int)(nh * B);
  dim3 grid((unsigned)(nqb * nhb));
#define UPIPE_DQ(C, R, P)                                                                  \
  hipLaunchKernelGGL((attn_bwd_dq_kernel<C, R, P>), grid, dim3(512), 0, st, Q, dO, lse_c, D, \
                     K, V, dQ, S, Sp, nh, h0, G, nqb, nhb, rope)
#define UPIPE_DQ_PARTS(C, R)             \
  if (parts == 1) UPIPE_DQ(C, R, 1);     \
  else if (parts == 2) UPIPE_DQ(C, R, 2); \
  else UPIPE_DQ(C, R, 4)
  if (causal) {
    if (rope.on) { UPIPE_DQ_PARTS(true, true); }
    else { UPIPE_DQ_PARTS(true, false); }
  } else {
    if (rope.on) { UPIPE_DQ_PARTS(false, true); }
    else { UPIPE_DQ_PARTS(false, false); }
  }
#undef UPIPE_DQ_PARTS
#undef UPIPE_DQ
  return hipGetLastError();
}

}  // namespace upipe
