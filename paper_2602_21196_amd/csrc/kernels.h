// Host-side launchers of the gfx950 kernels.  Every launcher enqueues on the
// given stream and returns the launch status; shapes are validated by the
// caller (api.cpp) before any of these run.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace upipe {

// Rows of 128 elements of several heads of a batch of sequences: element
// (b, s, h, e) is p[b * batch + s * row + h * head + e].  Token-major
// [B, S, H, d]: row = H d, head = d, batch = S H d; head-major [H, Sp, d]:
// row = d, head = Sp d.
struct HeadView {
  bf16* p;
  int64_t row, head, batch;
};

// ---- layout (layout.hip) -------------------------------------------------
// src [S, H, d] heads h0..h0+n-1  ->  dst [n, Sp, d]; rows >= S are zero.
hipError_t launch_pack_rows(const bf16* src, int64_t S, int H, int h0, int n,
                            int64_t Sp, bf16* dst, hipStream_t st);
// Rows s < S of src [n, Sp, d]  ->  heads h0..h0+n-1 of dst [S, H, d].
hipError_t launch_unpack_rows(const bf16* src, int64_t S, int H, int h0, int n,
                              int64_t Sp, bf16* dst, hipStream_t st);
// D[B, n, Sp] = rowsum(a * b) over the head width and lse_c[B, n, Sp] =
// -sqrt(d) times the rows of heads h0.. of lse [B, lse_heads, S]; zero for
// rows >= S.  Head hh of a and b is head h0 + hh.  B <= 65535.
hipError_t launch_rowdot_lse(const HeadView& a, const HeadView& b, const float* lse, int64_t S,
                             int64_t B, int lse_heads, int h0, int n, int64_t Sp, float* D,
                             float* lse_c, hipStream_t st);

// ---- attention forward (attn_fwd.hip) ------------------------------------
// The kernels address one head's rows with 32-bit byte offsets, up to the
// end of the last 128-row tile.
inline bool rows_addressable(int64_t S, int64_t row) {
  return round_up(S, SEQ_PAD) * row * 2 < (int64_t(1) << 32);
}
// Heads h0 .. h0 + nh - 1 of B sequences: Q, O (head u of the view is head
// h0 + u; they may be the same rows), K, V (head g of the view is key/value
// head g; rows_addressable) and lse [B, lse_heads, Sq].  Query row i sees
// key j iff j < Skv and (not causal or j <= i + delta); rows that see no key
// get O = 0, lse = -inf.  Self-attention: Sq = Skv = S, delta = 0.  `parts`
// as attn_fwd_key_parts says for the whole call's heads.
hipError_t launch_attn_fwd(const HeadView& Q, const HeadView& K, const HeadView& V,
                           const HeadView& O, float* lse, int64_t Sq, int64_t Skv, int64_t delta,
                           int64_t B, int lse_heads, int nh, int h0, int G, int causal, int parts,
                           hipStream_t st);
// Parts (1, 2 or 4) into which the waves of a workgroup split the keys of
// every stage, for a call over Hq heads.
int attn_fwd_key_parts(int64_t Sq, int64_t Skv, int64_t delta, int Hq, int causal);
// The same for few queries and many keys (one sequence, Sq <= 128), in two halves
// of the keys: side by side and then merged, their fp32 outputs in p0, p1, l0 and
// in O and lse (O is not Q then), or, without that room (p0 == nullptr), one after
// the other.  Both give the same bits.
struct FwdHalves {
  float* p0 = nullptr;     // [rows][128], rows = heads x Sq
  float* p1 = nullptr;     // [rows][64]
  float* l0 = nullptr;     // [rows]
  int stage = 0;           // the second half's first stage of 128 keys
};
// That stage, or 0 for calls that take their keys in one piece.
int attn_fwd_half_stage(int64_t Sq, int64_t Skv, int64_t delta, int causal);
// Halves of a call over nh heads, side by side if `room` holds their outputs.
FwdHalves attn_fwd_halves(int stage, int64_t Sq, int nh, char* room, size_t bytes);
hipError_t launch_attn_fwd_halves(const HeadView& Q, const HeadView& K, const HeadView& V,
                                  const HeadView& O, float* lse, int64_t Sq, int64_t Skv,
                                  int64_t delta, int lse_heads, int nh, int h0, int G, int causal,
                                  const FwdHalves& hv, hipStream_t st);
hipError_t launch_half_merge(const FwdHalves& hv, const HeadView& O, float* lse, int64_t Sq, int nh,
                             hipStream_t st);
// In place, per row (s, h) of o [S, H, d] and lse [H, S]: fold the partial
// result (o_p, lse_p) over a disjoint key set into (o, lse).
hipError_t launch_lse_merge(bf16* o, float* lse, const bf16* o_p,
                            const float* lse_p, int64_t S, int H,
                            hipStream_t st);

// ---- attention backward (attn_bwd.hip) -----------------------------------
// Rows u of lse_c and D [.][Sp] below belong to head h0 + u; lse_c holds
// -sqrt(d) lse, the initial value of a row's score accumulator (the kernels
// evaluate P = exp2(acc log2(e) / sqrt(d))).  Head u of Q, dO and dQ is head
// h0 + u, head g of K, V, dk, dv is key/value head g.
// Of one sequence: key/value gradients of the heads h0 .. h0 + nh - 1, accumulated in fp32 on top
// of dK32/dV32 [Hkv, Sp, d] (read unless the launch holds a group's first
// head; dK32 carries the unscaled sum with its sign flipped, -sum dS^T Q),
// written back there, or -- when the launch holds the group's last head --
// scaled and rounded into dk/dv.  The rows of Q and dO are rows_addressable,
// and as far apart in one as in the other.
hipError_t launch_attn_bwd_dkdv(const HeadView& Q, const HeadView& dO, const float* lse_c,
                                const float* D, const HeadView& K, const HeadView& V, float* dK32,
                                float* dV32, const HeadView& dk, const HeadView& dv, int64_t S,
                                int64_t Sp, int nh, int h0, int G, int causal, hipStream_t st);
// The same over every head of one sequence, with each key block's list of
// (head, query tile) cut into segments of T tiles that run side by side: their
// fp32 sums meet in slots of region0 (bytes0) and region1, both free until
// the call's last kernel is done.
struct DkdvSplit {
  int qs = 1;          // 128 / qs keys per workgroup
  int T = 0;           // tiles of a segment
  int whole = 0;       // segments of a key/value head that are not a list's last
  double est = 0;      // expected time, in tiles
};
struct DkdvSlots {
  float* p0 = nullptr;     // slots 0 .. n0 - 1
  float* p1 = nullptr;     // slots n0 ..
  int64_t n0 = 0;
  int T = 0, kv_heads = 1, whole = 0, per_head = 0;   // per_head: slots of a kv head
  __device__ float* at(int64_t i, int64_t floats) const {
    return i < n0 ? p0 + i * floats : p1 + (i - n0) * floats;
  }
};
// Segments for sequences of Sp padded rows, given what the regions hold.
DkdvSplit dkdv_split(int64_t Sp, int Hkv, int G, int causal, size_t bytes0, size_t bytes1);
hipError_t launch_attn_bwd_dkdv_split(const HeadView& Q, const HeadView& dO, const float* lse_c,
                                      const float* D, const HeadView& K, const HeadView& V,
                                      const HeadView& dk, const HeadView& dv, int64_t S, int64_t Sp,
                                      int Hkv, int G, int causal, const DkdvSplit& p, char* region0,
                                      size_t bytes0, char* region1, hipStream_t st);
// dQ of these heads of B sequences (rows b nh + u of lse_c and D); it may be
// the rows of Q or dO.  With rope.on, Q and K
// are the rotated ones and dQ is turned back by the inverse rotation of its
// row before it is rounded.  `parts` as attn_bwd_dq_key_parts says for the
// whole call's heads.  The rows of K and V are rows_addressable.
hipError_t launch_attn_bwd_dq(const HeadView& Q, const HeadView& dO, const float* lse_c,
                              const float* D, const HeadView& K, const HeadView& V,
                              const HeadView& dQ, int64_t S, int64_t Sp, int64_t B, int nh, int h0,
                              int G, int causal, int parts, RopeArgs rope, hipStream_t st);
// Parts (1, 2 or 4) into which the waves of a dQ workgroup split the keys of
// every stage, for a call over Hq heads.
int attn_bwd_dq_key_parts(int64_t S, int Hq, int causal);
// In place: rotate every head h < H of row s < S, the 128 values at element
// s * row + h * head of x, at position pos0 + s (inverse: by the opposite
// angle).  Token-major [S, H, d]: row = H * d, head = d.
hipError_t launch_rope(bf16* x, int64_t S, int H, int64_t row, int64_t head,
                       RopeArgs rope, int inverse, hipStream_t st);

}  // namespace upipe
