// Projection GEMMs of the attention block on gfx950: C = A . B, bf16 inputs,
// fp32 accumulation on MFMA 32x32x16.
//
// The block needs differently laid-out products (QKV projection, output
// projection, their data and weight gradients; paper Section 3.3 and
// Appendix A).  No tensor is transposed in HBM.  Every operand tile is staged
// into LDS as it lies in memory, 64 k at a time, by buffer->LDS copies (no
// register staging), and the MFMA fragments are read in one common k order,
// k = 8g + 0..7 within each 16-k step:
//   K-major operand  (k contiguous)    : rows = m (or n), 128 B of k each, two
//                                        rows to a 256-B LDS line; plain
//                                        16-byte reads;
//   MN-major operand (m/n contiguous)  : 128-wide column blocks of 64 lines of
//                                        256 B, line = k; transposing reads.
// Operands may be split into 128-wide blocks with their own stride (the
// head-major buffers [H][Sp][128]).
//
// Tiles (BM x BN per workgroup) by what bounds them: a CU's L2->LDS path (64
// B/clk) needs as long as its MFMAs for a 128 x 128 tile, half as long for 256 x
// 256.  So 256 x 256 wherever its tiles fill the chip, else 128 x 128 (256 x 128
// was never the fastest); two stages of 64 k each, the next one's copies in
// flight during the products.  Against 128 x 128 tiles of 128 k in one stage:
// 8192 x 4096 x 4096 272 -> 227 us (1011 -> 1210 TFLOP/s), 8192^3 1073 -> 884 us (1025 ->
// 1244).  A wave has 64 columns, 32 c + 64 nt + 0..31 of a 128-wide
// block (nt = 0, 1): the coordinate pairs (e, e + 64) of a head sit in one lane,
// which the rotary embedding of the head epilogue needs.  The k loop runs in
// ascending order with one fp32 accumulator chain per output element, so no
// result depends on the tile.
#include "common.h"
#include "gemm.h"

namespace upipe {

namespace {

constexpr int BK = 64;

// Address of operand element (r, k).
// The block width is a power of two (128, or the unblocked 2^50), so the
// block index and the offset inside it are a shift and a mask.
__device__ __forceinline__ const bf16* elem_ptr(const GemmOperand& o, bool kmajor, int64_t r,
                                                int64_t k) {
  const int sh = __builtin_ctzll((unsigned long long)o.blk);
  const int64_t mask = o.blk - 1;
  if (kmajor) return o.p + (k >> sh) * o.blk_stride + r * o.ld + (k & mask);
  return o.p + (r >> sh) * o.blk_stride + k * o.ld + (r & mask);
}

// Buffer resource of one wave's part of an operand tile at (r0, k0), as its four
// words: LINES lines of the tile (K-major: rows r0.. < rows_valid, 64 k of each;
// MN-major: k0.. < k_valid, the 128 columns from r0 on, none past rows_valid),
// so that padding reads as zero.
template <bool KMAJOR, int LINES>
__device__ __forceinline__ i32x4 tile_rsrc(const GemmOperand& o, int64_t r0, int64_t k0) {
  const int64_t valid = KMAJOR ? o.rows_valid - r0 : r0 < o.rows_valid ? o.k_valid - k0 : 0;
  const int64_t n = valid > LINES ? LINES : valid;
  const int64_t bytes = n <= 0 ? 0 : ((n - 1) * o.ld + (KMAJOR ? BK : 128)) * 2;
  return rsrc_words(elem_ptr(o, KMAJOR, r0, k0), (uint32_t)bytes);
}

// One operand's tile of R (m or n) x 64 k, R = 128 or 256, staged by W waves.
template <bool KMAJOR, int R, int W>
struct Tile {
  static constexpr int BYTES = R * BK * 2;
  static constexpr int NBLK = BYTES / 1024 / W;        // 1 KB blocks per wave
  static_assert(NBLK == 4, "copy4_b128");
  static constexpr int WAVES = W * 128 / R;            // that copy one 128-wide block
  uint32_t voff[NBLK];

  __device__ __forceinline__ void init(int64_t ld, int w, int lane) {
#pragma unroll
    for (int i = 0; i < NBLK; ++i) {
      if (KMAJOR) {
        // lines 4 blk.., line l = rows 2l, 2l + 1, chunk c of a row at c ^ (l & 7)
        const int blk = NBLK * w + i, line = 4 * blk + (lane >> 4), slot = lane & 15;
        const int row = 2 * line + (slot >> 3), c = (slot & 7) ^ (line & 7);
        voff[i] = (uint32_t)(row * ld * 2) + c * 16;
      } else {
        const int blk = NBLK * (w % WAVES) + i, line = 4 * blk + (lane >> 4);
        voff[i] = (uint32_t)(line * ld * 2) + (((lane & 15) ^ tsw(line)) << 4);
      }
    }
  }
  // This wave's copies of the tile at (r0, k0) to LDS address `lds`.
  __device__ __forceinline__ void issue(const GemmOperand& o, int64_t r0, int64_t k0, uint32_t lds,
                                        int w) const {
    const i32x4 r = tile_rsrc<KMAJOR, KMAJOR ? R : BK>(o, KMAJOR ? r0 : r0 + 128 * (w / WAVES), k0);
    copy4_b128(r, voff, 0, lds + NBLK * w * 1024);
  }
  // Per-lane base of the fragment reads of this wave's rows (m or n), from w0 on.
  static __device__ __forceinline__ uint32_t base(int w0, int lane) {
    const int r32 = lane & 31, g = lane >> 5, t = lane & 15, hi = (lane >> 4) & 1;
    if (KMAJOR)
      return w0 * 128 + (r32 >> 1) * 256 + ((((r32 & 1) << 3) | (g ^ ((r32 >> 1) & 7))) << 4);
    const uint32_t at = swzt(8 * g + (t >> 2), 2 * hi + ((t & 3) >> 1)) + ((t & 1) << 3);
    return (at ^ ((w0 & 127) * 2)) + (w0 >> 7) * (BK * 256);
  }
  // Fragment of the 32 rows r0.. (of the wave's; bits of r0 and w0 are apart) at
  // k-step ks (16 k): lane l gets row r0 + l % 32 at k = 16 ks + 8g + 0..7, g = l / 32.  MN-major: two
  // ds_read_b64_tr_b16 per lane; within each 16-lane group, loader lane t reads
  // the 8 bytes at line 16 ks + 8g + t/4 (+ 4 for the second read), columns r0 + 16
  // ((l >> 4) & 1) + 4 (t % 4); with the swzt swizzle the 8 lines x 4 chunks of one
  // read fill every bank exactly twice.
  static __device__ __forceinline__ bf16x8 frag(const char* smem, uint32_t at, int r0, int ks) {
    if (KMAJOR) return lds_read_b128(smem, (at ^ (32 * ks)) + r0 * 128);
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const uint32_t x = r0 * 2, k = ks * 4096;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(smem + (at ^ x) + k));
    const bf16x4 up =
        __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(smem + (at ^ (x + 16)) + k + 1024));
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = lo[e];
      v[4 + e] = up[e];
    }
    return v;
  }
};

// BM x BN = 256 x 256: eight waves of 128 x 64, one workgroup per CU; 128 x 128: four of
// 64 x 64, two workgroups per CU.  Two stages in LDS.
template <int BM, int BN>
struct Shape {
  static constexpr int WN = BN / 64, MT = BM / 64;
  static constexpr int WM = BM / (32 * MT), W = WM * WN;        // waves
  static constexpr int STAGE = (BM + BN) * BK * 2;
};

template <bool A_K, bool B_K, int EPI, int BM, int BN>
__global__ __launch_bounds__((64 * Shape<BM, BN>::W), 2) void gemm_kernel(
    GemmOperand A, GemmOperand B, GemmEpilogue E, int64_t M, int64_t N, int64_t k_len) {
  using H = Shape<BM, BN>;
  using TA = Tile<A_K, BM, H::W>;
  using TB = Tile<B_K, BN, H::W>;
  constexpr int MT = H::MT;
  __shared__ __attribute__((aligned(1024))) char smem[2 * H::STAGE];
  const uint32_t lds0 = lds_address(smem);
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r32 = lane & 31, g = lane >> 5;
  const int wm = w / H::WN, wn = w % H::WN;
  const int rowA = 32 * MT * wm;                                // of this wave in the tile
  const int colB = 128 * (wn >> 1) + 32 * (wn & 1);             // + 64 nt
  const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  // Workgroups go round-robin to the 8 XCDs, each with its own L2: every XCD
  // takes a contiguous run of (split, tile), the tiles of a split in bands of
  // eight along m, so that the ones running together share operand rows.
  int64_t tile, split;
  {
    const int64_t nx = gridDim.x, d = (int64_t)blockIdx.y * nx + blockIdx.x;
    const int64_t nwg = nx * gridDim.y, xcd = d % 8, per = nwg / 8, rem = nwg % 8;
    const int64_t L = xcd * per + (xcd < rem ? xcd : rem) + d / 8;
    tile = L % nx;
    split = L / nx;
  }
  const int64_t band = tile / (8 * tiles_n), in = tile % (8 * tiles_n);
  const int64_t bh = tiles_m - 8 * band < 8 ? tiles_m - 8 * band : 8;
  const int64_t m0 = (8 * band + in % bh) * BM, n0 = (in / bh) * BN;
  const int64_t kb0 = split * k_len;
  int64_t kend = kb0 + k_len;
  if (kend > E.k_total) kend = E.k_total;
  const int nk = kend > kb0 ? (int)((kend - kb0 + BK - 1) / BK) : 0;

  f32x16 acc[MT][2];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mt][nt][i] = 0.f;

  TA ta;
  TB tb;
  ta.init(A.ld, w, lane);
  tb.init(B.ld, w, lane);
  auto issue = [&](int kk) {
    const int64_t k0 = kb0 + (int64_t)kk * BK;
    const uint32_t at = lds0 + (kk & 1) * H::STAGE;
    ta.issue(A, m0, k0, at, w);
    tb.issue(B, n0, k0, at + TA::BYTES, w);
  };
  const uint32_t a_lane = TA::base(rowA, lane);
  const uint32_t b_lane = TA::BYTES + TB::base(colB, lane);
  if (nk > 0) issue(0);
  for (int kk = 0; kk < nk; ++kk) {
    // This wave's copies of stage kk have landed, its reads of stage kk - 1 are
    // done; past the barrier every wave's.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kk + 1 < nk) issue(kk + 1);
    const uint32_t aa = a_lane + (kk & 1) * H::STAGE, ba = b_lane + (kk & 1) * H::STAGE;
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 af[MT], bfr[2];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) af[mt] = TA::frag(smem, aa, 32 * mt, ks);
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) bfr[nt] = TB::frag(smem, ba, 64 * nt, ks);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) acc[mt][nt] = mfma32x32x16(af[mt], bfr[nt], acc[mt][nt]);
    }
    // Keep one k-step's fragment reads in flight ahead of the MFMAs (left to
    // itself the scheduler waits for a step's reads before its first MFMA:
    // 8192 x 4096 x 4096 -4 %).
    constexpr int NR = MT * (A_K ? 1 : 2) + 2 * (B_K ? 1 : 2);   // reads of a k-step
    constexpr int PER = (NR + 2 * MT - 1) / (2 * MT);             // per MFMA
    constexpr int NI = (3 * NR + PER - 1) / PER;
    __builtin_amdgcn_sched_group_barrier(0x100, NR, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, PER, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 8 * MT - NI, 0);
  }

  // ---- epilogues.  Lane holds column n0 + colB + 64 nt + r32 and rows
  //      m0 + rowA + 32 mt + 8a + 4g + b for element i = 4a + b.
  const int nb = (int)((n0 + colB) / 128);     // output head (HEADS)
  int grp = 0;
  if (EPI == GEMM_EPI_HEADS) {
    if (n0 + colB >= N) return;
    while (grp + 1 < E.n_groups && nb >= E.group[grp + 1].first) ++grp;
    if (E.rope.on && ((E.rope_groups >> grp) & 1)) {
      // Pair (e, e + 64) of rows m: acc[mt][0][i], acc[mt][1][i].  The turn of the
      // first row of each 32-row block is reduced in fp64; the offsets 8a + b
      // (< 28) add at most 28 theta_e / 2 pi turns in fp32.
      const double f = rope_turns_per_pos(32 * (wn & 1) + r32, E.rope.log2_base);
      const float ff = (float)f;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float t0 = rope_turn(E.rope.pos0 + m0 + rowA + 32 * mt + 4 * g, f);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          float c, s;
          cos_sin_turns(fmaf((float)(8 * (i >> 2) + (i & 3)), ff, t0), c, s);
          rope_pair(acc[mt][0], acc[mt][1], i, c, s, false);
        }
      }
    }
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const int64_t n = n0 + colB + 64 * nt + r32;
      const int64_t mb = m0 + rowA + 32 * mt + 4 * g;
      if (EPI != GEMM_EPI_HEADS && n >= N) continue;
      if (EPI == GEMM_EPI_HEADS) {
        const GemmEpilogue::Group& G = E.group[grp];
        bf16* dn = G.p + (nb - G.first) * G.head + n % 128;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int64_t m = mb + 8 * (i >> 2) + (i & 3);
          if (m < E.m_store) dn[m * G.row] = (bf16)acc[mt][nt][i];
        }
      } else if (EPI == GEMM_EPI_STORE) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int64_t m = mb + 8 * (i >> 2) + (i & 3);
          if (m < E.m_store) E.out[m * E.ldo + n] = (bf16)acc[mt][nt][i];
        }
      } else {  // GEMM_EPI_PARTIAL
        float* P = E.partial + split * M * N;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int64_t m = mb + 8 * (i >> 2) + (i & 3);
          if (m < M) P[m * N + n] = acc[mt][nt][i];
        }
      }
    }
}

// t = sum over splits s = 0.. of partial[s][m][n], summed in ascending s,
// then added to acc32[m][n] unless `first`; the total goes to acc32 unless
// `last`, else to out[m * ldo + n] as bf16.  HBM-bound: a thread has four
// consecutive columns (N is a multiple of 128).
__global__ __launch_bounds__(256) void reduce_splitk_kernel(const float* __restrict__ partial,
                                                            int splits, int64_t M, int64_t N,
                                                            bf16* __restrict__ out, int64_t ldo,
                                                            float* __restrict__ acc32,
                                                            int first, int last) {
  const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (idx >= M * N) return;
  f32x4 s = *reinterpret_cast<const f32x4*>(partial + idx);
  for (int k = 1; k < splits; ++k)
    s += *reinterpret_cast<const f32x4*>(partial + (int64_t)k * M * N + idx);
  if (!first) s = *reinterpret_cast<const f32x4*>(acc32 + idx) + s;
  if (last) {
    const int64_t m = idx / N, n = idx % N;
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (bf16)s[e];
    *reinterpret_cast<bf16x4*>(out + m * ldo + n) = v;
  } else {
    *reinterpret_cast<f32x4*>(acc32 + idx) = s;
  }
}

template <bool A_K, bool B_K, int EPI, int BM, int BN>
hipError_t launch_t(const GemmOperand& A, const GemmOperand& B, const GemmEpilogue& E, int64_t M,
                    int64_t N, int64_t k_len, int splits, hipStream_t st) {
  dim3 grid((unsigned)(((M + BM - 1) / BM) * ((N + BN - 1) / BN)), (unsigned)splits);
  hipLaunchKernelGGL((gemm_kernel<A_K, B_K, EPI, BM, BN>), grid, dim3(64 * Shape<BM, BN>::W), 0, st,
                     A, B, E, M, N, k_len);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm(const GemmOperand& A, bool a_kmajor, const GemmOperand& B, bool b_kmajor,
                       const GemmEpilogue& E, int epi, int64_t M, int64_t N, int64_t k_len,
                       int splits, hipStream_t st) {
  // A K-major tile reads 64 consecutive k of each row: the k range must be
  // made of whole tiles (an MN-major operand is bounded by its buffer
  // resource instead); pieces must start on tile boundaries.
  if ((M % 128) || (N % 128) || (k_len % 128)) return hipErrorInvalidValue;
  if ((a_kmajor || b_kmajor) && (E.k_total % 128)) return hipErrorInvalidValue;
  // Rounds on 256 CUs: a 256 x 256 tile takes 0.8 of four 128 x 128 ones, two of
  // which run side by side (us, 128 | 256: 8192 x 4096 x 4096 252 | 231; 8192^3 1087 | 892;
  // 65536 x 1280 x 5120 907 | 785; 16384 x 640 x 512 22.2 | 21.6; 8192 x 768 x 4096, 96
  // large tiles, 56 | 90; 3072 x 2048 x 1024 20 | 30).  No result depends on it.
  const int64_t big = ((M + 255) / 256) * ((N + 255) / 256) * splits;
  const int64_t small = (M / 128) * (N / 128) * splits;
  const bool large = 1.6 * ((big + 255) / 256) < (small + 511) / 512;
#define UPIPE_GEMM_CASE(AK, BK_, EP)                                                            \
  if (a_kmajor == AK && b_kmajor == BK_ && epi == EP)                                           \
    return large ? launch_t<AK, BK_, EP, 256, 256>(A, B, E, M, N, k_len, splits, st)            \
                 : launch_t<AK, BK_, EP, 128, 128>(A, B, E, M, N, k_len, splits, st);
  UPIPE_GEMM_CASE(true, false, GEMM_EPI_HEADS)     // X . Wqkv
  UPIPE_GEMM_CASE(true, false, GEMM_EPI_STORE)     // O . Wo
  UPIPE_GEMM_CASE(true, true, GEMM_EPI_HEADS)      // dY . Wo^T
  UPIPE_GEMM_CASE(true, true, GEMM_EPI_STORE)      // dQKV . Wqkv^T
  UPIPE_GEMM_CASE(false, false, GEMM_EPI_PARTIAL)  // X^T . dQKV, O^T . dY
#undef UPIPE_GEMM_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_reduce_splitk(const float* partial, int splits, int64_t M, int64_t N, bf16* out,
                                int64_t ldo, float* acc32, int first, int last, hipStream_t st) {
  const int64_t n = M * N;
  hipLaunchKernelGGL(reduce_splitk_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, st,
                     partial, splits, M, N, out, ldo, acc32, first, last);
  return hipGetLastError();
}

}  // namespace upipe
