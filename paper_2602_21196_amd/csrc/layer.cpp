// Attention-block entry points: projections around the attention of all heads.
//
// The paper runs stages of U heads (Section 3.3) because every stage's heads
// arrive by an all-to-all.  On one GPU all heads are here, so each product over
// heads runs once and the attention kernels take all heads in one launch; no
// result depends on U.
// Forward (Appendix A "Untied Ulysses (forward)"):
//   Q | K | V = x Wqkv                     one product; Q in the rows of
//                                          o_saved, K and V head-major
//   final_out = attention(Q, K, V)         in the place of Q, lse saved
//   y = final_out Wo                       output projection
// Backward (Appendix A "Untied Ulysses (backward)"), with Q, K, V
// recomputed from x (activation checkpointing keeps x, final_out, lse):
//   Q | K | V = x Wqkv                     Q in the dQ part of dQKV
//   dFO   = dY Wo^T                        gradient of final_out, head-major
//   (O, lse = attention(Q, K, V))          full checkpointing only: the
//                                          attention output was not kept
//   dWo   = final_out^T dY                 split-K over S, ordered sum
//   D     = rowsum(dFO * O)
//   dK, dV, then dQ in the place of Q      attention backward
//   dx    = [dQ | dK | dV] Wqkv^T          one product, bf16 out
//   dWqkv = x^T [dQ | dK | dV]             split-K over S
// Against the products and attention of one chunk of U heads at a time, 8192 tokens
// of the Llama3-8B share (d_model 4096, 4 heads, U = 1): the five QKV products
// 2 x 307 -> 2 x 95 us.
// Where o_saved lies over x or wqkv the forward runs the chunks of U heads (K and
// V first, then a chunk's Q and attention at a time).
// Rotary embedding (optional, Section 4 "Implementation"): Q and K are
// rotated in the projection epilogue, on the fp32 accumulators, before they
// are rounded and stored -- in place, with no extra pass or fp32 copy.  The
// backward recomputes them the same way and turns dQ back by the inverse
// rotation in the dQ kernel's final write, and dK in one in-place pass.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/upipe.h"
#include "api_internal.h"
#include "gemm.h"
#include "kernels.h"

namespace upipe {

namespace {

int check_layer_shape(int64_t S, int d_model, int Hq, int Hkv, int d, int U) {
  int rc = check_attn_shape(S, Hq, Hkv, d, U);
  if (rc != UPIPE_OK) return rc;
  if (d_model < 1) return UPIPE_ERR_INVALID_ARG;
  if (d_model % 128 != 0) return UPIPE_ERR_UNSUPPORTED;
  if (d_model > 65536) return UPIPE_ERR_UNSUPPORTED;
  if (round_up(S, SEQ_PAD) * (int64_t)d_model >= (int64_t(1) << 40)) return UPIPE_ERR_UNSUPPORTED;
  return UPIPE_OK;
}

// Split length of the sequence for the weight gradient of a [M, N] weight: a
// function of S and the whole weight only (never of U), a multiple of 256.
// The pieces that cost least: rounds of 256 x 256 tiles on 256 CUs against tiles,
// plus the write and read of a piece's fp32 partial, as long as the product
// over 1200 rows (4096 x 768, 8192 rows: 32 pieces 116 + 124 us for product and
// sum, 5 pieces 60 + 12).
int64_t wgrad_split_len(int64_t S, int64_t M, int64_t N) {
  const int64_t tiles = ((M + 255) / 256) * ((N + 255) / 256);
  int64_t best = 1;
  double best_cost = 0;
  for (int64_t s = 1; s <= 32; ++s) {
    const int64_t rounds = (tiles * s + 255) / 256;
    const double cost = rounds * 256.0 / (tiles * s) + 1200.0 * s / S;
    if (s == 1 || cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return std::max<int64_t>(256, round_up((S + best - 1) / best, 256));
}

struct LayerFwdPlan {
  int64_t Sp = 0;
  size_t Kp = 0, Vp = 0;
  size_t Qc = 0;       // a chunk's queries, where o_saved overlaps x or wqkv
  size_t total = 0;
};

struct LayerBwdPlan {
  int64_t Sp = 0;
  bool carry = false;          // a key/value group spans several chunks
  int o_heads = 0;             // heads of recomputed attention output held at a time
  size_t Kp = 0, Vp = 0, dK32 = 0, dV32 = 0, D = 0, lse_c = 0;
  size_t Oc = 0, lse_r = 0;    // recomputed attention output (full checkpointing)
  size_t dFO = 0, dQKV = 0;
  size_t scratch = 0, scratch_bytes = 0;   // split-K partials; dK/dV segment sums
  size_t dWqkv32 = 0, dWo32 = 0;   // weight-gradient sums over a batch of sequences
  size_t total = 0;
};

LayerFwdPlan plan_layer_fwd(int64_t S, int d_model, int Hq, int Hkv, int U) {
  (void)d_model;
  (void)Hq;
  LayerFwdPlan p;
  p.Sp = round_up(S, SEQ_PAD);
  const size_t head = (size_t)p.Sp * HEAD_DIM * 2;
  Carver c;
  p.Kp = c.take(Hkv * head);
  p.Vp = c.take(Hkv * head);
  p.Qc = c.take(U * head);
  c.take(U * head);     // in the size that callers have been told to bring; unused
  p.total = c.used;
  return p;
}

// Bytes of the backward's workspace when the weight gradients were cut into up
// to 32 pieces and a chunk's Q, O and rows were held: callers have been told to
// bring these, and the plan below stays within them: up to 32 of fewer, longer
// pieces, and the D and lse rows of up to 64 heads are 512 bytes a row of the
// sequence, where a chunk's buffers (U >= 1) were 520.
size_t layer_bwd_budget(int64_t S, int d_model, int Hq, int Hkv, int U) {
  const int64_t Sp = round_up(S, SEQ_PAD);
  const int64_t len = std::max<int64_t>(256, round_up((S + 31) / 32, 256));
  const size_t head = (size_t)Sp * HEAD_DIM * 2;
  const int64_t widest = (int64_t)(Hq + 2 * Hkv) * HEAD_DIM;
  Carver c;
  c.take(2 * Hkv * head);
  if (group_split(Hq, Hkv, U)) c.take(4 * Hkv * head);
  c.take(2 * U * head);
  c.take(2 * (size_t)U * Sp * 4);
  c.take((size_t)Hq * S * 4);
  c.take((2 * Hq + 2 * Hkv) * head);
  c.take((size_t)((S + len - 1) / len) * d_model * widest * 4);
  c.take((size_t)d_model * widest * 4);
  c.take((size_t)Hq * HEAD_DIM * d_model * 4);
  return c.used;
}

LayerBwdPlan plan_layer_bwd(int64_t S, int d_model, int Hq, int Hkv, int U) {
  LayerBwdPlan p;
  p.Sp = round_up(S, SEQ_PAD);
  const size_t head = (size_t)p.Sp * HEAD_DIM * 2;
  const size_t rows = (size_t)Hq * p.Sp * 4;
  const int64_t nqkv = (int64_t)(Hq + 2 * Hkv) * HEAD_DIM, qw = (int64_t)Hq * HEAD_DIM;
  Carver c;
  p.Kp = c.take(Hkv * head);
  p.Vp = c.take(Hkv * head);
  p.carry = group_split(Hq, Hkv, U);
  if (p.carry) {
    p.dK32 = c.take(Hkv * head * 2);
    p.dV32 = c.take(Hkv * head * 2);
  }
  p.D = c.take(rows);
  p.lse_c = c.take(rows);
  p.lse_r = c.take((size_t)Hq * S * 4);
  p.dFO = c.take(Hq * head);
  p.dQKV = c.take((Hq + 2 * Hkv) * head);
  const int64_t l1 = wgrad_split_len(S, d_model, nqkv), l2 = wgrad_split_len(S, qw, d_model);
  p.scratch_bytes = std::max((size_t)((S + l1 - 1) / l1) * d_model * nqkv * 4,
                             (size_t)((S + l2 - 1) / l2) * d_model * qw * 4);
  p.scratch = c.take(p.scratch_bytes);
  p.dWqkv32 = c.take((size_t)d_model * nqkv * 4);
  p.dWo32 = c.take((size_t)qw * d_model * 4);
  // Recomputed attention output: in the rest of the budget, or, where that
  // holds fewer heads (at 40 heads and U = 1 it may hold none), in the dK | dV
  // part of dQKV, which is written after the last of them is done with.
  const size_t budget = layer_bwd_budget(S, d_model, Hq, Hkv, U);
  const size_t used = c.used + 256;
  const int rest = budget > used ? (int)std::min<size_t>(Hq, (budget - used) / head) : 0;
  p.o_heads = std::min(Hq, 2 * Hkv);
  p.Oc = p.dQKV + Hq * head;
  if (rest > p.o_heads) {
    p.o_heads = rest;
    p.Oc = c.take(rest * head);
  }
  p.total = std::max(c.used, budget);
  return p;
}

// Head-major [heads][Sp][128] output from p on.
GemmEpilogue heads_epi(bf16* p, int64_t Sp, int64_t m_store) {
  GemmEpilogue e{};
  e.group[0] = {p, HEAD_DIM, Sp * HEAD_DIM, 0};
  e.n_groups = 1;
  e.m_store = m_store;
  return e;
}

// Q | K | V of a product with Wqkv: Q wherever its view says, K and V
// head-major, Q and K rotated.
GemmEpilogue qkv_epi(const HeadView& Q, bf16* Kp, bf16* Vp, int Hq, int Hkv, int64_t S, int64_t Sp,
                     RopeArgs rope) {
  GemmEpilogue e{};
  e.group[0] = {Q.p, Q.row, Q.head, 0};
  e.group[1] = {Kp, HEAD_DIM, Sp * HEAD_DIM, Hq};
  e.group[2] = {Vp, HEAD_DIM, Sp * HEAD_DIM, Hq + Hkv};
  e.n_groups = 3;
  e.m_store = S;
  e.rope = rope;
  e.rope_groups = rope.on ? 3 : 0;
  return e;
}

// bf16 result rows m < m_store into out[m * ldo + n].
GemmEpilogue store_epi(bf16* out, int64_t ldo, int64_t m_store) {
  GemmEpilogue e{};
  e.out = out;
  e.ldo = ldo;
  e.m_store = m_store;
  return e;
}

// C = A . B over the whole k range in one piece.
hipError_t gemm1(const GemmOperand& A, bool ak, const GemmOperand& B, bool bk, GemmEpilogue E,
                 int epi, int64_t M, int64_t N, int64_t K, hipStream_t st) {
  E.k_total = K;
  return launch_gemm(A, ak, B, bk, E, epi, M, N, round_up(K, 128), 1, st);
}

}  // namespace

// One sequence of the batch.
int run_layer_fwd_seq(const bf16* x, const bf16* wqkv, const bf16* wo, bf16* y, bf16* o_saved,
                      float* lse, int64_t S, int dm, int Hq, int Hkv, int U, RopeArgs rope,
                      char* ws, hipStream_t st) {
  const LayerFwdPlan p = plan_layer_fwd(S, dm, Hq, Hkv, U);
  const int64_t Sp = p.Sp, nqkv = (int64_t)(Hq + 2 * Hkv) * HEAD_DIM;
  const int64_t qw = (int64_t)Hq * HEAD_DIM;
  bf16* Kp = (bf16*)(ws + p.Kp);
  bf16* Vp = (bf16*)(ws + p.Vp);
  const HeadView QO = token_major(o_saved, S, Hq), K = head_major(Kp, Sp), V = head_major(Vp, Sp);
  const GemmOperand X = operand(x, dm, S, dm);
  const int G = Hq / Hkv, parts = attn_fwd_key_parts(S, S, 0, Hq, 1);
  const int64_t o_bytes = S * qw * 2;
  if (!overlap(o_saved, o_bytes, x, S * dm * 2) && !overlap(o_saved, o_bytes, wqkv, dm * nqkv * 2)) {
    UPIPE_LAUNCH(kGemm, st,
                 gemm1(X, true, operand(wqkv, nqkv, nqkv, dm), false,
                       qkv_epi(QO, Kp, Vp, Hq, Hkv, S, Sp, rope), GEMM_EPI_HEADS, Sp, nqkv, dm, st));
    UPIPE_LAUNCH(kAttnFwd, st,
                 launch_attn_fwd(QO, K, V, QO, lse, S, S, 0, 1, Hq, Hq, 0, G, 1, parts, st));
  } else {
    // The queries cannot pass through o_saved while x and wqkv are read: K and V
    // first, then chunks of U heads, each writing o_saved when its queries are
    // formed.
    const int64_t kvw = 2 * (int64_t)Hkv * HEAD_DIM, w = (int64_t)U * HEAD_DIM;
    const HeadView Qc = head_major((bf16*)(ws + p.Qc), Sp);
    UPIPE_LAUNCH(kGemm, st,
                 gemm1(X, true, operand(wqkv + qw, nqkv, kvw, dm), false,
                       qkv_epi(Qc, Kp, Vp, 0, Hkv, S, Sp, rope), GEMM_EPI_HEADS, Sp, kvw, dm, st));
    for (int h0 = 0; h0 < Hq; h0 += U) {
      UPIPE_LAUNCH(kGemm, st,
                   gemm1(X, true, operand(wqkv + (int64_t)h0 * HEAD_DIM, nqkv, w, dm), false,
                         qkv_epi(Qc, Kp, Vp, U, Hkv, S, Sp, rope), GEMM_EPI_HEADS, Sp, w, dm, st));
      UPIPE_LAUNCH(kAttnFwd, st,
                   launch_attn_fwd(Qc, K, V, sub(QO, 0, h0), lse, S, S, 0, 1, Hq, U, h0, G, 1, parts,
                                   st));
    }
  }
  // y = final_out Wo.
  UPIPE_LAUNCH(kGemm, st,
               gemm1(operand(o_saved, qw, S, qw), true, operand(wo, dm, dm, qw), false,
                     store_epi(y, dm, S), GEMM_EPI_STORE, Sp, dm, qw, st));
  return UPIPE_OK;
}

// One sequence of the batch: dx of the sequence; the weight gradients of
// the sequence are added to the fp32 sums unless `first` and rounded into
// dwqkv, dwo when `last`.
int run_layer_bwd_seq(const bf16* x, const bf16* wqkv, const bf16* wo, const bf16* o_saved,
                      const float* lse, const bf16* dy, bf16* dx, bf16* dwqkv, bf16* dwo,
                      int64_t S, int dm, int Hq, int Hkv, int U, RopeArgs rope, int first,
                      int last, char* ws, hipStream_t st) {
  const LayerBwdPlan p = plan_layer_bwd(S, dm, Hq, Hkv, U);
  const int64_t Sp = p.Sp, nqkv = (int64_t)(Hq + 2 * Hkv) * HEAD_DIM;
  const int64_t qw = (int64_t)Hq * HEAD_DIM;
  const int64_t head = Sp * HEAD_DIM;   // elements of one head-major head
  bf16* Kp = (bf16*)(ws + p.Kp);
  bf16* Vp = (bf16*)(ws + p.Vp);
  float* D = (float*)(ws + p.D);
  float* lse_c = (float*)(ws + p.lse_c);
  bf16* dFO = (bf16*)(ws + p.dFO);
  bf16* dQKV = (bf16*)(ws + p.dQKV);     // heads: dQ 0..Hq-1, dK Hq.., dV Hq+Hkv..
  bf16* dKh = dQKV + (int64_t)Hq * head;
  bf16* dVh = dKh + (int64_t)Hkv * head;
  const int G = Hq / Hkv;
  const HeadView Q = head_major(dQKV, Sp), K = head_major(Kp, Sp), V = head_major(Vp, Sp);
  const HeadView dO = head_major(dFO, Sp);
  const GemmOperand X = operand(x, dm, S, dm);
  const GemmOperand XT = operand(x, dm, dm, S);        // MN-major view: (m = col, k = s)
  const GemmOperand dY = operand(dy, dm, S, dm);
  const GemmOperand dYn = operand(dy, dm, dm, S);      // MN-major view: (n = col, k = s)

  // Weight gradient C[M][N] = sum over s of A(m, s) B(n, s), split into fixed
  // pieces of the sequence and summed in order (then onto the batch sum
  // acc32 [M][N]) into out[m * ldo + n].
  auto wgrad = [&](const GemmOperand& A, const GemmOperand& B, int64_t M, int64_t N, int64_t len,
                   bf16* out, int64_t ldo, size_t acc32) -> int {
    GemmEpilogue e{};
    e.partial = (float*)(ws + p.scratch);
    e.k_total = S;
    const int splits = (int)((S + len - 1) / len);
    UPIPE_LAUNCH(kGemmWgrad, st,
                 launch_gemm(A, false, B, false, e, GEMM_EPI_PARTIAL, M, N, len, splits, st));
    UPIPE_LAUNCH(kReduceSplitk, st,
                 launch_reduce_splitk(e.partial, splits, M, N, out, ldo, (float*)(ws + acc32), first,
                                      last, st));
    return UPIPE_OK;
  };

  // Q, K and V again (Q and K rotated); dQ will take the place of Q.
  UPIPE_LAUNCH(kGemm, st,
               gemm1(X, true, operand(wqkv, nqkv, nqkv, dm), false,
                     qkv_epi(Q, Kp, Vp, Hq, Hkv, S, Sp, rope), GEMM_EPI_HEADS, Sp, nqkv, dm, st));
  // dFO = dY Wo^T for every head (Wo rows are k-contiguous).
  UPIPE_LAUNCH(kGemm, st,
               gemm1(dY, true, operand(wo, dm, qw, dm), true, heads_epi(dFO, Sp, S),
                     GEMM_EPI_HEADS, Sp, qw, dm, st));
  const int64_t wo_len = wgrad_split_len(S, qw, dm);
  int rc;
  if (o_saved != nullptr) {   // dWo = final_out^T dY from the kept final_out
    rc = wgrad(operand(o_saved, qw, qw, S), dYn, qw, dm, wo_len, dwo, dm, p.dWo32);
    if (rc != UPIPE_OK) return rc;
    UPIPE_LAUNCH(kRowdotLse, st,
                 launch_rowdot_lse(dO, token_major(o_saved, S, Hq), lse, S, 1, Hq, 0, Hq, Sp, D,
                                   lse_c, st));
  } else {
    // Full checkpointing: the attention output and lse again (the same kernel
    // on the same operands: bitwise what the forward produced), and their
    // rows of dWo, as many heads at a time as the workspace holds.
    float* lse_r = (float*)(ws + p.lse_r);
    bf16* Oc = (bf16*)(ws + p.Oc);
    const int parts = attn_fwd_key_parts(S, S, 0, Hq, 1);
    for (int h0 = 0; h0 < Hq; h0 += p.o_heads) {
      const int n = std::min(p.o_heads, Hq - h0);
      const int64_t w = (int64_t)n * HEAD_DIM, row0 = (int64_t)h0 * HEAD_DIM * dm;
      const HeadView O = head_major(Oc, Sp);
      UPIPE_LAUNCH(kAttnFwd, st,
                   launch_attn_fwd(sub(Q, 0, h0), K, V, O, lse_r, S, S, 0, 1, Hq, n, h0, G, 1,
                                   parts, st));
      UPIPE_LAUNCH(kRowdotLse, st,
                   launch_rowdot_lse(sub(dO, 0, h0), O, lse_r, S, 1, Hq, h0, n, Sp, D + h0 * Sp,
                                     lse_c + h0 * Sp, st));
      rc = wgrad(operand(Oc, HEAD_DIM, w, S, HEAD_DIM, head), dYn, w, dm, wo_len, dwo + row0, dm,
                 p.dWo32 + row0 * 4);
      if (rc != UPIPE_OK) return rc;
    }
  }
  // The weight gradients' scratch is free now: dK/dV segment sums.
  if (S < kPerHeadRows) {
    const DkdvSplit cut = dkdv_split(Sp, Hkv, G, 1, p.scratch_bytes, 0);
    UPIPE_LAUNCH(kAttnBwdDkdv, st,
                 launch_attn_bwd_dkdv_split(Q, dO, lse_c, D, K, V, head_major(dKh, Sp),
                                            head_major(dVh, Sp), S, Sp, Hkv, G, 1, cut,
                                            ws + p.scratch, p.scratch_bytes, nullptr, st));
  } else {
    float* dK32 = p.carry ? (float*)(ws + p.dK32) : nullptr;
    float* dV32 = p.carry ? (float*)(ws + p.dV32) : nullptr;
    rc = run_dkdv(Q, dO, lse_c, D, K, V, dK32, dV32, head_major(dKh, Sp), head_major(dVh, Sp), S,
                  Sp, Hq, 0, G, 1, st);
    if (rc != UPIPE_OK) return rc;
  }
  UPIPE_LAUNCH(kAttnBwdDq, st,
               launch_attn_bwd_dq(Q, dO, lse_c, D, K, V, Q, S, Sp, 1, Hq, 0, G, 1,
                                  attn_bwd_dq_key_parts(S, Hq, 1), rope, st));
  // dK is the gradient with respect to the rotated keys: turn it back, in
  // place (one bf16 pass over [Hkv, S, d]; kept out of the dK/dV kernel,
  // whose register allocation is at its limit).
  if (rope.on)
    UPIPE_LAUNCH(kRope, st, launch_rope(dKh, S, Hkv, HEAD_DIM, head, rope, 1, st));
  // dx = [dQ | dK | dV] Wqkv^T (head-major A; Wqkv rows are k-contiguous).
  UPIPE_LAUNCH(kGemm, st,
               gemm1(operand(dQKV, HEAD_DIM, S, nqkv, HEAD_DIM, head), true,
                     operand(wqkv, nqkv, dm, nqkv), true, store_epi(dx, dm, S), GEMM_EPI_STORE,
                     Sp, dm, nqkv, st));
  // dWqkv = x^T [dQ | dK | dV].
  return wgrad(XT, operand(dQKV, HEAD_DIM, nqkv, S, HEAD_DIM, head), dm, nqkv,
               wgrad_split_len(S, dm, nqkv), dwqkv, nqkv, p.dWqkv32);
}

// Batches: the B sequences run one after another through the same
// workspace; only the caller's tensors grow with B.
int run_layer_fwd(const bf16* x, const bf16* wqkv, const bf16* wo, bf16* y, bf16* o_saved,
                  float* lse, int64_t B, int64_t S, int dm, int Hq, int Hkv, int U, RopeArgs rope,
                  char* ws, hipStream_t st) {
  const int64_t xs = S * dm, os = S * Hq * HEAD_DIM, ls = (int64_t)Hq * S;
  for (int64_t b = 0; b < B; ++b) {
    const int rc = run_layer_fwd_seq(x + b * xs, wqkv, wo, y + b * xs, o_saved + b * os,
                                     lse + b * ls, S, dm, Hq, Hkv, U, rope, ws, st);
    if (rc != UPIPE_OK) return rc;
  }
  return UPIPE_OK;
}

int run_layer_bwd(const bf16* x, const bf16* wqkv, const bf16* wo, const bf16* o_saved,
                  const float* lse, const bf16* dy, bf16* dx, bf16* dwqkv, bf16* dwo, int64_t B,
                  int64_t S, int dm, int Hq, int Hkv, int U, RopeArgs rope, char* ws,
                  hipStream_t st) {
  const int64_t xs = S * dm, os = S * Hq * HEAD_DIM, ls = (int64_t)Hq * S;
  const bool kept = o_saved != nullptr;
  for (int64_t b = 0; b < B; ++b) {
    const int rc = run_layer_bwd_seq(x + b * xs, wqkv, wo, kept ? o_saved + b * os : nullptr,
                                     kept ? lse + b * ls : nullptr, dy + b * xs, dx + b * xs,
                                     dwqkv, dwo, S, dm, Hq, Hkv, U, rope, b == 0, b == B - 1, ws,
                                     st);
    if (rc != UPIPE_OK) return rc;
  }
  return UPIPE_OK;
}

}  // namespace upipe

using namespace upipe;

extern "C" {

size_t upipe_layer_fwd_workspace_size(int64_t S, int d_model, int Hq, int Hkv, int d, int U) {
  if (check_layer_shape(S, d_model, Hq, Hkv, d, U) != UPIPE_OK) return 0;
  return plan_layer_fwd(S, d_model, Hq, Hkv, U).total;
}

size_t upipe_layer_bwd_workspace_size(int64_t S, int d_model, int Hq, int Hkv, int d, int U) {
  if (check_layer_shape(S, d_model, Hq, Hkv, d, U) != UPIPE_OK) return 0;
  return plan_layer_bwd(S, d_model, Hq, Hkv, U).total;
}

int upipe_layer_fwd_ex(const void* x, const void* wqkv, const void* wo, void* y, void* o_saved,
                       float* lse_saved, int64_t B, int64_t S, int d_model, int Hq, int Hkv,
                       int d, int U, double rope_base, int64_t pos0, void* ws,
                       size_t ws_bytes, hipStream_t stream) {
  try {
    int rc = check_layer_shape(S, d_model, Hq, Hkv, d, U);
    if (rc != UPIPE_OK) return rc;
    if (!batch_ok(B, S * std::max<int64_t>(d_model, (int64_t)Hq * HEAD_DIM)))
      return UPIPE_ERR_INVALID_ARG;
    RopeArgs rope;
    rc = make_rope(rope_base, pos0, S, &rope);
    if (rc != UPIPE_OK) return rc;
    if (!aligned16(x) || !aligned16(wqkv) || !aligned16(wo) || !aligned16(y) ||
        !aligned16(o_saved) || !aligned16(lse_saved) || !aligned16(ws))
      return UPIPE_ERR_INVALID_ARG;
    if (ws_bytes < plan_layer_fwd(S, d_model, Hq, Hkv, U).total) return UPIPE_ERR_WORKSPACE;
    return run_layer_fwd((const bf16*)x, (const bf16*)wqkv, (const bf16*)wo, (bf16*)y,
                         (bf16*)o_saved, lse_saved, B, S, d_model, Hq, Hkv, U, rope, (char*)ws,
                         stream);
  } catch (...) {
    return UPIPE_ERR_HIP;
  }
}

int upipe_layer_bwd_ex(const void* x, const void* wqkv, const void* wo, const void* o_saved,
                       const float* lse_saved, const void* dy, void* dx, void* dwqkv,
                       void* dwo, int64_t B, int64_t S, int d_model, int Hq, int Hkv, int d,
                       int U, double rope_base, int64_t pos0, void* ws, size_t ws_bytes,
                       hipStream_t stream) {
  try {
    int rc = check_layer_shape(S, d_model, Hq, Hkv, d, U);
    if (rc != UPIPE_OK) return rc;
    if (!batch_ok(B, S * std::max<int64_t>(d_model, (int64_t)Hq * HEAD_DIM)))
      return UPIPE_ERR_INVALID_ARG;
    RopeArgs rope;
    rc = make_rope(rope_base, pos0, S, &rope);
    if (rc != UPIPE_OK) return rc;
    // o_saved and lse_saved: both given (kept attention output), or both NULL
    // (full checkpointing: recomputed).
    if ((o_saved == nullptr) != (lse_saved == nullptr)) return UPIPE_ERR_INVALID_ARG;
    const bool kept = o_saved != nullptr;
    if (!aligned16(x) || !aligned16(wqkv) || !aligned16(wo) || (kept && !aligned16(o_saved)) ||
        (kept && !aligned16(lse_saved)) || !aligned16(dy) || !aligned16(dx) ||
        !aligned16(dwqkv) || !aligned16(dwo) || !aligned16(ws))
      return UPIPE_ERR_INVALID_ARG;
    if (ws_bytes < plan_layer_bwd(S, d_model, Hq, Hkv, U).total) return UPIPE_ERR_WORKSPACE;
    return run_layer_bwd((const bf16*)x, (const bf16*)wqkv, (const bf16*)wo,
                         (const bf16*)o_saved, lse_saved, (const bf16*)dy, (bf16*)dx,
                         (bf16*)dwqkv, (bf16*)dwo, B, S, d_model, Hq, Hkv, U, rope, (char*)ws,
                         stream);
  } catch (...) {
    return UPIPE_ERR_HIP;
  }
}

int upipe_gemm_bf16(const void* a, const void* b, void* c, int64_t M, int64_t N, int64_t K,
                    hipStream_t stream) {
  try {
    if (M < 1 || N < 1 || K < 1) return UPIPE_ERR_INVALID_ARG;
    if (M % 128 || N % 128 || K % 128) return UPIPE_ERR_UNSUPPORTED;
    if (M > 65536 || N > 65536 || K > 65536) return UPIPE_ERR_UNSUPPORTED;
    if (!aligned16(a) || !aligned16(b) || !aligned16(c)) return UPIPE_ERR_INVALID_ARG;
    // A [M, K] row-major is K-major; B [K, N] row-major is N-major.
    UPIPE_LAUNCH(kGemm, stream,
                 gemm1(operand((const bf16*)a, K, M, K), true, operand((const bf16*)b, N, N, K),
                       false, store_epi((bf16*)c, N, M), GEMM_EPI_STORE, M, N, K, stream));
    return UPIPE_OK;
  } catch (...) {
    return UPIPE_ERR_HIP;
  }
}

int upipe_layer_fwd(const void* x, const void* wqkv, const void* wo, void* y, void* o_saved,
                    float* lse_saved, int64_t S, int d_model, int Hq, int Hkv, int d, int U,
                    void* ws, size_t ws_bytes, hipStream_t stream) {
  return upipe_layer_fwd_ex(x, wqkv, wo, y, o_saved, lse_saved, 1, S, d_model, Hq, Hkv, d, U,
                            0.0, 0, ws, ws_bytes, stream);
}

int upipe_layer_bwd(const void* x, const void* wqkv, const void* wo, const void* o_saved,
                    const float* lse_saved, const void* dy, void* dx, void* dwqkv, void* dwo,
                    int64_t S, int d_model, int Hq, int Hkv, int d, int U, void* ws,
                    size_t ws_bytes, hipStream_t stream) {
  return upipe_layer_bwd_ex(x, wqkv, wo, o_saved, lse_saved, dy, dx, dwqkv, dwo, 1, S, d_model,
                            Hq, Hkv, d, U, 0.0, 0, ws, ws_bytes, stream);
}

}  // extern "C"
