// Shared device-side helpers for the gfx950 kernels.
//
// MFMA fragment conventions used throughout (v_mfma_f32_32x32x16_bf16, wave64):
//   A operand: lane l supplies row (l % 32) of the 32x16 A tile and the 8
//              k-values of k-group g = l / 32.
//   B operand: lane l supplies column (l % 32) of the 16x32 B tile and the 8
//              k-values of k-group g.
//   The k-values a lane supplies may be any fixed permutation of the 16 k's
//   as long as A and B use the same one; contractions only need agreement.
//   C/D:       lane l holds column (l % 32); element i of its 16 floats is
//              row 8*(i/4) + 4*g + (i%4).
//
// Transposed operands (V^T, K^T, Q^T, dO^T) are never stored: they are read
// out of the row-major [S][128] tiles in LDS with ds_read_b64_tr_b16 (see
// tr_operand), which hands each lane one column of a 4-row block.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace upipe {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int HEAD_DIM = 128;   // the only supported head width
constexpr int SEQ_PAD = 128;    // sequence padding granule of packed buffers

__host__ __device__ inline int64_t round_up(int64_t x, int64_t m) {
  return (x + m - 1) / m * m;
}

__device__ __forceinline__ f32x16 mfma32x32x16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float fast_exp2(float x) {
  return __builtin_amdgcn_exp2f(x);
}

__device__ __forceinline__ bf16x8 lds_read_b128(const char* base, uint32_t off) {
  return *reinterpret_cast<const bf16x8*>(base + off);
}

// Buffer -> LDS copy of 16 bytes per lane (buffer_load_dwordx4 ... lds): the
// bytes at voff + soff (lane offset + uniform offset) of lane L land at LDS
// address lds + 16 * L, zeros where that offset is past the resource's bytes.  No
// vector ALU work for the address; tracked by vmcnt.  Written out, because the
// kernels issue the copies of a later tile
// between reads of this one: the compiler cannot tell which LDS bytes a copy
// writes, and would wait for it before the next transposing read.  The wave
// waits itself (wait_vmem, then a barrier) before the bytes are read, and no
// one reads or writes them meanwhile.  A buffer instruction may read an SGPR
// only five wait states after a vector instruction (a readlane, say, of one
// that was spilled) wrote it; the compiler does not look into the text, so the
// wait is in it, once for up to four copies (one by one it cost the 8192^3
// product 861 against 851 us and the dK/dV walks 3 %).  No register results;
// `lds` is an LDS address (lds_address).  m0 is not in the clobber lists: the
// compiler reserves it, warns of such an entry and does not act on it.  It holds
// no value there between these texts as long as the kernels use none of the
// instructions that take it (tests/test_build.py looks through the assembly).
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4 rsrc_words(const void* base, uint32_t bytes) {
  const uint64_t a = (uint64_t)base;
  return i32x4{(int)a, (int)((a >> 32) & 0xffff), (int)bytes, 0x00020000};
}
__device__ __forceinline__ void copy_b128(i32x4 r, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds), "v"(voff), "s"(r), "s"(soff));
}
// Four copies to consecutive 1 KB blocks.
__device__ __forceinline__ void copy4_b128(i32x4 r, const uint32_t (&voff)[4], uint32_t soff,
                                           uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %5, %6 offen lds\n\t"
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %5, %6 offen lds\n\t"
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %3, %5, %6 offen lds\n\t"
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %4, %5, %6 offen lds"
      :: "s"(lds), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(r), "s"(soff)
      : "scc");
}
// Two copies from each of two sources, to consecutive 1 KB blocks at lds and at
// lds + GAP.
template <int GAP>
__device__ __forceinline__ void copy2x2_b128(i32x4 r0, i32x4 r1, uint32_t voff0, uint32_t voff1,
                                             uint32_t soff, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %3, %5 offen lds\n\t"
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, %5 offen lds\n\t"
      "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %4, %5 offen lds\n\t"
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %4, %5 offen lds"
      :: "s"(lds), "v"(voff0), "v"(voff1), "s"(r0), "s"(r1), "s"(soff), "n"(GAP - 1024)
      : "scc");
}
__device__ __forceinline__ uint32_t lds_address(const char* p) {
  typedef __attribute__((address_space(3))) const char lds_char;
  return (uint32_t)(uintptr_t)(lds_char*)p;
}

// Wait until every outstanding global load of this wave has completed.
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x3F70); }

// 16-byte chunk swizzles of 256-B rows (16 chunks).  swz256: chunk c of row
// r at c ^ (r & 15).  swzt: chunk c of row r at c ^ tsw(r), where tsw swaps
// the two 2-bit halves of r mod 16.  Both put the sixteen consecutive rows of
// a plain MFMA operand read (same logical chunk) in sixteen distinct slots;
// swzt also spreads the 8 rows x 4 chunks of a transposing read (tr_operand)
// over every slot exactly twice, the minimum for its 512 bytes.
__device__ __forceinline__ uint32_t swz256(int r, int c) { return r * 256 + ((c ^ (r & 15)) << 4); }
__device__ __forceinline__ uint32_t tsw(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
__device__ __forceinline__ uint32_t swzt(int r, int c) { return r * 256 + ((c ^ tsw(r)) << 4); }

// MFMA operand whose k index runs down the rows of a row-major [k][n] tile of
// 256-B rows stored with swzt (A and B operands have the same lane layout):
// lane l gets column n0 + (l % 32) at rows k0 + 4g + {0..3} (elements 0..3)
// and k0 + 8 + 4g + {0..3} (elements 4..7), g = l / 32 -- the k order in
// which a lane holds the rows of a C tile (rows 8a + 4g + b), so P and dS
// fragments taken from C tiles pair with it directly.  ds_read_b64_tr_b16:
// within each 16-lane group, loader lane t reads the 8 bytes at row
// k0 + 4g + t/4, columns n0 + 16 * ((l >> 4) & 1) + 4 (t % 4), and receiver
// lane t gets column t of the group's 16 columns for those four rows.
__device__ __forceinline__ bf16x8 tr_operand(const char* tile, int k0, int n0, int lane) {
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  const int t = lane & 15, hi = (lane >> 4) & 1, g = lane >> 5;
  const int col = n0 + 16 * hi + 4 * (t & 3);
  const int r0 = k0 + 4 * g + (t >> 2);
  const uint32_t cb = (uint32_t)(col & 7) << 1;   // byte offset inside the 16-byte chunk
  const bf16x4 lo =
      __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(tile + swzt(r0, col >> 3) + cb));
  const bf16x4 up =
      __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(tile + swzt(r0 + 8, col >> 3) + cb));
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = lo[e];
    v[4 + e] = up[e];
  }
  return v;
}

// The same addresses as one per-lane base and exclusive-ors, for kernels that
// cannot hold one register per address: with base = swz(r, g), chunk 2s + g of
// the row (s < 8) lies at base ^ 32 s and rows 32 on at + 8192 (swz256 and
// swzt alike); a transposing read's columns 32 dt on at tr_base ^ 64 dt, rows
// 16 on at + 4096, and its upper half (8 rows on) at tr_base ^ 32, + 2048.
__device__ __forceinline__ uint32_t tr_base(int lane) {
  const int t = lane & 15, hi = (lane >> 4) & 1, g = lane >> 5;
  return swzt(4 * g + (t >> 2), 2 * hi + ((t & 3) >> 1)) + ((t & 1) << 3);
}
// Columns 32 dt.., rows k0.. (a multiple of 16) of the tile whose tr_base,
// with the tile's offset added, is `tb`.
__device__ __forceinline__ bf16x8 tr_operand_at(const char* smem, uint32_t tb, int k0, int dt) {
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  const uint32_t lo_at = (tb ^ (64 * dt)) + k0 * 256, up_at = (tb ^ (64 * dt + 32)) + k0 * 256 + 2048;
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(smem + lo_at));
  const bf16x4 up = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(smem + up_at));
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = lo[e];
    v[4 + e] = up[e];
  }
  return v;
}

// ---- rotary position embedding (RoFormer), head coordinate pairs (e, e + 64)
// for e < 64: at sequence position p the pair turns by p * theta_e with
// theta_e = base^(-e/64); the inverse (transpose) turns by the opposite angle.
struct RopeArgs {
  double log2_base;   // log2 of the frequency base
  int64_t pos0;       // position of sequence row 0
  int on;             // 0: no rotation
};

// theta_e / (2 pi): turns per position of pair e, in fp64.  Positions reach
// 2^24, so the whole turns of p * theta_e are removed in fp64 before anything
// is rounded to fp32.
__device__ __forceinline__ double rope_turns_per_pos(int e, double log2_base) {
  return exp2(-(double)e * log2_base * (1.0 / 64.0)) * 0.15915494309189535;
}

// Fractional part, in [-1/2, 1/2], of p * f turns.
__device__ __forceinline__ float rope_turn(int64_t p, double f) {
  const double r = (double)p * f;
  return (float)(r - rint(r));
}

// cos(2 pi t), sin(2 pi t): v_cos_f32 / v_sin_f32 take their argument in
// turns; t is first brought into [-1/2, 1/2].
__device__ __forceinline__ void cos_sin_turns(float t, float& c, float& s) {
  t -= rintf(t);
  c = __builtin_amdgcn_cosf(t);
  s = __builtin_amdgcn_sinf(t);
}

// Rotate the pair (a, b) by the angle whose cos / sin are (c, s); `inverse`
// turns the other way.
__device__ __forceinline__ void rope_pair(float& a, float& b, float c, float s, bool inverse) {
  if (inverse) s = -s;
  const float ra = a * c - b * s;
  const float rb = b * c + a * s;
  a = ra;
  b = rb;
}

// The same on element i of two accumulator tiles.
__device__ __forceinline__ void rope_pair(f32x16& a, f32x16& b, int i, float c, float s,
                                          bool inverse) {
  float x = a[i], y = b[i];
  rope_pair(x, y, c, s, inverse);
  a[i] = x;
  b[i] = y;
}

}  // namespace upipe
