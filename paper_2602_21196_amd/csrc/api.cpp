// C ABI of the head-chunked attention library (declared in include/upipe.h).
//
// Host-side responsibilities: argument validation before anything is
// enqueued, the workspace plan, the route of a call (all heads in place in one
// launch; or, for dK/dV from 65536 rows on and wherever an output overlaps an
// input, the chunks of U heads of UPipe, paper Section 3.3, through one
// chunk-sized set of buffers), and optional per-kernel event timing.  All
// kernels run on the caller's stream.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <cmath>

#include <mutex>
#include <new>
#include <vector>

#include "../../include/upipe.h"
#include "api_internal.h"
#include "kernels.h"

namespace upipe {

// ------------------------------------------------------------ profiling
namespace {

struct ProfRecord {
  int family;
  hipEvent_t start, stop;
};

struct Profiler {
  bool on = false;
  std::vector<ProfRecord> recs;
  std::vector<hipEvent_t> pool;
  hipEvent_t get() {
    if (!pool.empty()) {
      hipEvent_t e = pool.back();
      pool.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
};

Profiler& prof() {
  static Profiler p;
  return p;
}

}  // namespace

const char* const kFamilyNames[] = {
    "pack_rows",      "unpack_rows",   "rowdot_lse",     "attn_fwd",
    "attn_bwd_dkdv",  "attn_bwd_dq",   "gemm",           "gemm_wgrad",
    "reduce_splitk",  "lse_merge",     "rope",           "split_merge",
};
const int kNumFamilies = sizeof(kFamilyNames) / sizeof(kFamilyNames[0]);

ProfScope::ProfScope(int family, hipStream_t st) : st_(st) {
  Profiler& p = prof();
  if (!p.on) return;
  start_ = p.get();
  stop_ = p.get();
  family_ = family;
  if (start_ && stop_) (void)hipEventRecord(start_, st_);
}

ProfScope::~ProfScope() {
  Profiler& p = prof();
  if (!p.on || !start_ || !stop_) return;
  (void)hipEventRecord(stop_, st_);
  try {
    p.recs.push_back({family_, start_, stop_});
  } catch (...) {
  }
}

// --------------------------------------------------------------- checks
bool aligned16(const void* p) { return p && ((uintptr_t)p & 15u) == 0; }

int check_attn_shape(int64_t S, int Hq, int Hkv, int d, int U) {
  if (S < 1 || Hq < 1 || Hkv < 1 || U < 1) return UPIPE_ERR_INVALID_ARG;
  if (Hq % Hkv != 0 || Hq % U != 0) return UPIPE_ERR_INVALID_ARG;
  if (d != HEAD_DIM) return UPIPE_ERR_UNSUPPORTED;
  if (Hq > kMaxHeads) return UPIPE_ERR_UNSUPPORTED;
  const int64_t Sp = round_up(S, SEQ_PAD);
  if (Sp > kMaxSeq) return UPIPE_ERR_UNSUPPORTED;
  if (Sp * (int64_t)Hq * d >= (int64_t(1) << 40)) return UPIPE_ERR_UNSUPPORTED;
  return UPIPE_OK;
}

bool group_split(int Hq, int Hkv, int U) {
  const int G = Hq / Hkv;
  for (int g = 0; g < Hkv; ++g)
    if ((g * G) / U != ((g + 1) * G - 1) / U) return true;
  return false;
}

// ----------------------------------------------------------- ws planning
size_t Carver::take(size_t bytes) {
  const size_t off = (used + 255) & ~size_t(255);
  used = off + bytes;
  return off;
}

AttnFwdPlan plan_attn_fwd_ring(int64_t Sq, int64_t Skv, int Hq, int Hkv, int U) {
  AttnFwdPlan p;
  p.Sp = round_up(Sq, SEQ_PAD);
  p.Skvp = round_up(Skv, SEQ_PAD);
  const size_t qhead = (size_t)p.Sp * HEAD_DIM * 2, kvhead = (size_t)p.Skvp * HEAD_DIM * 2;
  Carver c;
  if (!kv_in_place(Skv, Hkv)) {
    p.Kp = c.take(Hkv * kvhead);
    p.Vp = c.take(Hkv * kvhead);
  }
  // The size that callers have been told to bring.  Kp and Vp are used where
  // the keys and values cannot be read in place, Qc, Oc and lse_part where an
  // output overlaps an input.  (Up to 32768 rows there is room for two outputs
  // and lse rows, of a key range split in halves; one of them is used.)
  p.ns = p.Sp <= 128 * 256 && p.Skvp >= 256 ? 2 : 1;
  p.Qc = c.take(U * qhead);
  p.Oc = c.take(p.ns * U * qhead);
  if (p.ns > 1) p.lse_part = c.take((size_t)p.ns * U * p.Sp * 4);
  p.total = c.used;
  return p;
}

AttnFwdPlan plan_attn_fwd(int64_t S, int Hq, int Hkv, int U) {
  return plan_attn_fwd_ring(S, S, Hq, Hkv, U);
}

AttnBwdPlan plan_attn_bwd(int64_t S, int Hq, int Hkv, int U) {
  AttnBwdPlan p;
  p.Sp = round_up(S, SEQ_PAD);
  const size_t head = (size_t)p.Sp * HEAD_DIM * 2;
  const size_t row32 = (size_t)p.Sp * 4;
  Carver c;
  p.kv_direct = kv_in_place(S, Hkv);
  if (!p.kv_direct) {
    p.Kp = c.take(Hkv * head);
    p.Vp = c.take(Hkv * head);
  }
  p.carry = group_split(Hq, Hkv, U);
  if (p.carry) {
    p.dK32 = c.take(Hkv * head * 2);
    p.dV32 = c.take(Hkv * head * 2);
  }
  p.Qc = c.take(U * head);
  p.dOc = c.take(U * head);
  // D and lse rows: of a chunk, or, in the room of its dQ too where that is
  // written in place, of all heads
  p.rows = c.take(U * head);
  c.take(U * row32);
  c.take(U * row32);
  p.total = c.used;
  return p;
}

// ------------------------------------------------------- attention paths
// Token-major [B, S, H, d].
HeadView token_major(const bf16* p, int64_t S, int H) {
  return HeadView{const_cast<bf16*>(p), (int64_t)H * HEAD_DIM, HEAD_DIM, S * H * HEAD_DIM};
}

// Head-major [H, Sp, d] (one sequence).
HeadView head_major(const bf16* p, int64_t Sp) {
  return HeadView{const_cast<bf16*>(p), HEAD_DIM, Sp * HEAD_DIM, 0};
}

// Sequence b, head u (from the view's first) of a view, and of [B][.][Sp] rows.
HeadView sub(HeadView x, int64_t b, int64_t u) {
  x.p += b * x.batch + u * x.head;
  return x;
}

int run_dkdv(const HeadView& Q, const HeadView& dO, const float* lse_c, const float* D,
             const HeadView& K, const HeadView& V, float* dK32, float* dV32, const HeadView& dk,
             const HeadView& dv, int64_t S, int64_t Sp, int nh, int h0, int G, int causal,
             hipStream_t st) {
  const int step = dK32 != nullptr || G == 1 ? 1 : nh;
  for (int u = 0; u < nh; u += step)
    UPIPE_LAUNCH(kAttnBwdDkdv, st,
                 launch_attn_bwd_dkdv(sub(Q, 0, u), sub(dO, 0, u), lse_c + u * Sp, D + u * Sp, K, V,
                                      dK32, dV32, dk, dv, S, Sp, step, h0 + u, G, causal, st));
  return UPIPE_OK;
}

int run_attn_fwd_ring(const bf16* q, const bf16* k, const bf16* v, bf16* o, float* lse, int64_t B,
                      int64_t Sq, int64_t Skv, int64_t delta, int Hq, int Hkv, int causal,
                      int U, char* ws, hipStream_t st) {
  const int G = Hq / Hkv;
  const int parts = attn_fwd_key_parts(Sq, Skv, delta, Hq, causal);
  const HeadView Q = token_major(q, Sq, Hq), O = token_major(o, Sq, Hq);
  const HeadView K = token_major(k, Skv, Hkv), V = token_major(v, Skv, Hkv);
  // Whether the outputs may be written while others still read the inputs.  o
  // may be q itself: a workgroup reads its queries before it writes them.
  const int64_t q_bytes = B * Q.batch * 2, kv_bytes = B * K.batch * 2;
  const int64_t lse_bytes = B * Hq * Sq * 4;
  const bool apart = (o == q || !overlap(o, q_bytes, q, q_bytes)) &&
                     !overlap(o, q_bytes, k, kv_bytes) && !overlap(o, q_bytes, v, kv_bytes) &&
                     !overlap(lse, lse_bytes, q, q_bytes) &&
                     !overlap(lse, lse_bytes, k, kv_bytes) && !overlap(lse, lse_bytes, v, kv_bytes);
  const AttnFwdPlan p = plan_attn_fwd_ring(Sq, Skv, Hq, Hkv, U);
  // All heads of one sequence, or a chunk of them.
  const int stage = B == 1 ? attn_fwd_half_stage(Sq, Skv, delta, causal) : 0;
  auto attend = [&](const HeadView& Qb, const HeadView& Kb, const HeadView& Vb, const HeadView& Ob,
                    float* rows, int nh, int h0, char* room, size_t room_bytes) -> int {
    if (stage == 0) {
      UPIPE_LAUNCH(kAttnFwd, st,
                   launch_attn_fwd(Qb, Kb, Vb, Ob, rows, Sq, Skv, delta, 1, Hq, nh, h0, G, causal,
                                   parts, st));
      return UPIPE_OK;
    }
    const FwdHalves hv = attn_fwd_halves(stage, Sq, nh, Ob.p != Qb.p ? room : nullptr, room_bytes);
    UPIPE_LAUNCH(kAttnFwd, st,
                 launch_attn_fwd_halves(Qb, Kb, Vb, Ob, rows, Sq, Skv, delta, Hq, nh, h0, G, causal,
                                        hv, st));
    if (hv.p0 != nullptr)
      UPIPE_LAUNCH(kSplitMerge, st,
                   launch_half_merge(hv, Ob, rows + (int64_t)h0 * Sq, Sq, nh, st));
    return UPIPE_OK;
  };
  if (rows_addressable(Skv, K.row) && apart) {
    if (stage > 0) return attend(Q, K, V, O, lse, Hq, 0, ws, p.total);
    // Every tensor in place, all heads of as many sequences as one grid holds.
    const int64_t per_seq = (Sq * parts + 255) / 256 * Hq;
    const int64_t nb = std::max<int64_t>(1, (int64_t(1) << 22) / per_seq);
    for (int64_t b = 0; b < B; b += nb) {
      UPIPE_LAUNCH(kAttnFwd, st,
                   launch_attn_fwd(sub(Q, b, 0), sub(K, b, 0), sub(V, b, 0), sub(O, b, 0),
                                   lse + b * Hq * Sq, Sq, Skv, delta, std::min(nb, B - b), Hq, Hq,
                                   0, G, causal, parts, st));
    }
    return UPIPE_OK;
  }
  // Token-major key/value rows of one head span 2^32 bytes or more, or an
  // output overlaps an input: pack keys and values head-major (unless they lie
  // so), one sequence after another.  With an overlap nothing may be read after
  // the first write, so chunks of U heads go through the workspace: a chunk's
  // queries are packed, its outputs written back when it is done.
  bf16* Kp = (bf16*)(ws + p.Kp);
  bf16* Vp = (bf16*)(ws + p.Vp);
  bf16* Qc = (bf16*)(ws + p.Qc);
  bf16* Oc = (bf16*)(ws + p.Oc);
  for (int64_t b = 0; b < B; ++b) {
    HeadView Kb = sub(K, b, 0), Vb = sub(V, b, 0);
    float* lse_b = lse + b * Hq * Sq;
    if (!kv_in_place(Skv, Hkv)) {
      UPIPE_LAUNCH(kPackRows, st, launch_pack_rows(Kb.p, Skv, Hkv, 0, Hkv, p.Skvp, Kp, st));
      UPIPE_LAUNCH(kPackRows, st, launch_pack_rows(Vb.p, Skv, Hkv, 0, Hkv, p.Skvp, Vp, st));
      Kb = head_major(Kp, p.Skvp);
      Vb = head_major(Vp, p.Skvp);
    }
    if (apart) {
      const int rc = attend(sub(Q, b, 0), Kb, Vb, sub(O, b, 0), lse_b, Hq, 0, ws + p.Qc,
                            p.total - p.Qc);
      if (rc != UPIPE_OK) return rc;
      continue;
    }
    for (int h0 = 0; h0 < Hq; h0 += U) {
      float* to = lse_b + (int64_t)h0 * Sq;      // the chunk's lse rows
      float* rows = p.ns > 1 ? (float*)(ws + p.lse_part) : to;
      UPIPE_LAUNCH(kPackRows, st, launch_pack_rows(sub(Q, b, 0).p, Sq, Hq, h0, U, p.Sp, Qc, st));
      // The kernel counts lse rows from head 0 on.
      const int rc = attend(head_major(Qc, p.Sp), Kb, Vb, head_major(Oc, p.Sp),
                            rows - (int64_t)h0 * Sq, U, h0, nullptr, 0);
      if (rc != UPIPE_OK) return rc;
      UPIPE_LAUNCH(kUnpackRows, st,
                   launch_unpack_rows(Oc, Sq, Hq, h0, U, p.Sp, sub(O, b, 0).p, st));
      if (rows != to)
        UPIPE_LAUNCH(kUnpackRows, st,
                     hipMemcpyAsync(to, rows, (size_t)U * Sq * 4, hipMemcpyDeviceToDevice, st));
    }
  }
  return UPIPE_OK;
}

int make_rope(double base, int64_t pos0, int64_t S, RopeArgs* out) {
  *out = RopeArgs{0.0, 0, 0};
  if (base == 0.0) return UPIPE_OK;
  if (!(base > 0.0) || !std::isfinite(base)) return UPIPE_ERR_INVALID_ARG;
  if (pos0 < 0 || pos0 > kMaxRopePos || S > kMaxRopePos - pos0) return UPIPE_ERR_UNSUPPORTED;
  *out = RopeArgs{std::log2(base), pos0, 1};
  return UPIPE_OK;
}

int run_attn_fwd(const bf16* q, const bf16* k, const bf16* v, bf16* o,
                 float* lse, int64_t B, int64_t S, int Hq, int Hkv, int causal, int U,
                 char* ws, hipStream_t st) {
  return run_attn_fwd_ring(q, k, v, o, lse, B, S, S, 0, Hq, Hkv, causal, U, ws, st);
}

int run_attn_bwd(const bf16* q, const bf16* k, const bf16* v, const bf16* o,
                 const float* lse, const bf16* dout, bf16* dq, bf16* dk,
                 bf16* dv, int64_t B, int64_t S, int Hq, int Hkv, int causal, int U,
                 char* ws, hipStream_t st) {
  const AttnBwdPlan p = plan_attn_bwd(S, Hq, Hkv, U);
  const int G = Hq / Hkv;
  const int parts = attn_bwd_dq_key_parts(S, Hq, causal);
  const HeadView Q = token_major(q, S, Hq), O = token_major(o, S, Hq);
  const HeadView dO = token_major(dout, S, Hq), dQ = token_major(dq, S, Hq);
  const HeadView K = token_major(k, S, Hkv), V = token_major(v, S, Hkv);
  const HeadView dK = token_major(dk, S, Hkv), dV = token_major(dv, S, Hkv);
  const int64_t rows = Hq * p.Sp;                        // D and lse rows of a sequence
  const size_t row_bytes = (size_t)rows * 8;
  const int64_t q_bytes = B * Q.batch * 2, kv_bytes = B * K.batch * 2;
  bool apart = true;     // outputs from the inputs that are read after a first write
  for (const bf16* in : {q, dout, o})
    apart = apart && !overlap(dq, q_bytes, in, q_bytes) && !overlap(dk, kv_bytes, in, q_bytes) &&
            !overlap(dv, kv_bytes, in, q_bytes);
  for (const bf16* in : {k, v})
    apart = apart && !overlap(dq, q_bytes, in, kv_bytes) && !overlap(dk, kv_bytes, in, kv_bytes) &&
            !overlap(dv, kv_bytes, in, kv_bytes);

  static_assert(kPerHeadRows * kMaxHeads * HEAD_DIM * 2 < (int64_t(1) << 32),
                "rows below kPerHeadRows are rows_addressable");
  if (S < kPerHeadRows && apart) {
    // Every tensor in place.  dK/dV of all heads of a sequence in one launch,
    // cut into segments that run side by side: their slots lie behind the
    // rows and in dq, which is written last.  Cut for the smallest workspace
    // that a chunk size of this call could bring, so that no sum depends on U
    // (nor on the batch).
    size_t least = p.total;
    for (int u = 1; u <= Hq; ++u)
      if (Hq % u == 0) least = std::min(least, plan_attn_bwd(S, Hq, Hkv, u).total);
    auto cut_beside = [&](int64_t seqs) {
      return dkdv_split(p.Sp, Hkv, G, causal, least - seqs * row_bytes, (size_t)Q.batch * 2);
    };
    // The rows of four sequences, whose dQ then runs in one launch, unless
    // their room is worth more to the segments.
    int64_t nb = 1;
    DkdvSplit cut = cut_beside(1);
    if (4 * row_bytes <= least) {
      const DkdvSplit four = cut_beside(4);
      if (four.est <= 1.03 * cut.est) {
        nb = 4;
        cut = four;
      }
    }
    const size_t taken = nb * row_bytes;
    for (int64_t b0 = 0; b0 < B; b0 += nb) {
      const int64_t n = std::min(nb, B - b0);
      float* D = (float*)ws;
      float* lse_c = D + n * rows;
      UPIPE_LAUNCH(kRowdotLse, st,
                   launch_rowdot_lse(sub(dO, b0, 0), sub(O, b0, 0), lse + b0 * Hq * S, S, n, Hq, 0,
                                     Hq, p.Sp, D, lse_c, st));
      for (int64_t b = b0; b < b0 + n; ++b)
        UPIPE_LAUNCH(kAttnBwdDkdv, st,
                     launch_attn_bwd_dkdv_split(
                         sub(Q, b, 0), sub(dO, b, 0), lse_c + (b - b0) * rows, D + (b - b0) * rows,
                         sub(K, b, 0), sub(V, b, 0), sub(dK, b, 0), sub(dV, b, 0), S, p.Sp, Hkv, G,
                         causal, cut, ws + taken, p.total - taken, (char*)sub(dQ, b, 0).p, st));
      UPIPE_LAUNCH(kAttnBwdDq, st,
                   launch_attn_bwd_dq(sub(Q, b0, 0), sub(dO, b0, 0), lse_c, D, sub(K, b0, 0),
                                      sub(V, b0, 0), sub(dQ, b0, 0), S, p.Sp, n, Hq, 0, G, causal,
                                      parts, RopeArgs{}, st));
    }
    return UPIPE_OK;
  }

  // Long sequences: dK/dV of one head fills the chip, and walks its Q and dO
  // rows 1 - 3.5 % faster where they are packed (measured before its copies went
  // out between products, 131072 rows of 4 heads 33.4 against 34.6 ms; rows 1 KB
  // apart use 4 of an L2's 16 channels).  So chunks
  // of U heads are packed for it, and dQ takes all heads in place after the
  // last one, if the rows of all heads fit behind the packed ones.
  // Where an output overlaps an input (any length), nothing of a chunk may be
  // read after its first write: its dQ comes from the packed rows too, and goes
  // through the workspace.
  float* dK32 = p.carry ? (float*)(ws + p.dK32) : nullptr;
  float* dV32 = p.carry ? (float*)(ws + p.dV32) : nullptr;
  bf16* Qc = (bf16*)(ws + p.Qc);
  bf16* dOc = (bf16*)(ws + p.dOc);
  bf16* dQc = (bf16*)(ws + p.rows);      // overlap only
  const size_t dq_bytes = apart ? 0 : (size_t)U * p.Sp * HEAD_DIM * 2;
  const bool keep_rows = apart && p.total - p.rows >= row_bytes;
  const int64_t n_rows = (keep_rows ? Hq : U) * p.Sp;
  float* D = (float*)(ws + p.rows + dq_bytes);
  float* lse_c = D + n_rows;
  const bool kv_pack = !p.kv_direct && (!rows_addressable(S, K.row) || !apart);
  for (int64_t b = 0; b < B; ++b) {
    HeadView Kb = sub(K, b, 0), Vb = sub(V, b, 0);
    if (kv_pack) {
      bf16* Kp = (bf16*)(ws + p.Kp);
      bf16* Vp = (bf16*)(ws + p.Vp);
      UPIPE_LAUNCH(kPackRows, st, launch_pack_rows(Kb.p, S, Hkv, 0, Hkv, p.Sp, Kp, st));
      UPIPE_LAUNCH(kPackRows, st, launch_pack_rows(Vb.p, S, Hkv, 0, Hkv, p.Sp, Vp, st));
      Kb = head_major(Kp, p.Sp);
      Vb = head_major(Vp, p.Sp);
    }
    for (int h0 = 0; h0 < Hq; h0 += U) {
      float* Dh = D + (keep_rows ? h0 * p.Sp : 0);
      float* lh = lse_c + (keep_rows ? h0 * p.Sp : 0);
      UPIPE_LAUNCH(kPackRows, st, launch_pack_rows(sub(Q, b, 0).p, S, Hq, h0, U, p.Sp, Qc, st));
      UPIPE_LAUNCH(kPackRows, st, launch_pack_rows(sub(dO, b, 0).p, S, Hq, h0, U, p.Sp, dOc, st));
      UPIPE_LAUNCH(kRowdotLse, st,
                   launch_rowdot_lse(sub(dO, b, h0), sub(O, b, h0), lse + b * Hq * S, S, 1, Hq, h0,
                                     U, p.Sp, Dh, lh, st));
      const int rc = run_dkdv(head_major(Qc, p.Sp), head_major(dOc, p.Sp), lh, Dh, Kb, Vb, dK32,
                              dV32, sub(dK, b, 0), sub(dV, b, 0), S, p.Sp, U, h0, G, causal, st);
      if (rc != UPIPE_OK) return rc;
      if (!apart) {
        UPIPE_LAUNCH(kAttnBwdDq, st,
                     launch_attn_bwd_dq(head_major(Qc, p.Sp), head_major(dOc, p.Sp), lh, Dh, Kb, Vb,
                                        head_major(dQc, p.Sp), S, p.Sp, 1, U, h0, G, causal, parts,
                                        RopeArgs{}, st));
        UPIPE_LAUNCH(kUnpackRows, st,
                     launch_unpack_rows(dQc, S, Hq, h0, U, p.Sp, sub(dQ, b, 0).p, st));
        continue;
      }
      const int d0 = keep_rows ? 0 : h0, nh = keep_rows ? Hq : U;
      if (d0 + nh == h0 + U)
        UPIPE_LAUNCH(kAttnBwdDq, st,
                     launch_attn_bwd_dq(sub(Q, b, d0), sub(dO, b, d0), lse_c, D, Kb, Vb,
                                        sub(dQ, b, d0), S, p.Sp, 1, nh, d0, G, causal, parts,
                                        RopeArgs{}, st));
    }
  }
  return UPIPE_OK;
}

}  // namespace upipe

using namespace upipe;

extern "C" {

const char* upipe_status_string(int status) {
  switch (status) {
    case UPIPE_OK: return "UPIPE_OK";
    case UPIPE_ERR_INVALID_ARG: return "UPIPE_ERR_INVALID_ARG";
    case UPIPE_ERR_UNSUPPORTED: return "UPIPE_ERR_UNSUPPORTED";
    case UPIPE_ERR_WORKSPACE: return "UPIPE_ERR_WORKSPACE";
    case UPIPE_ERR_HIP: return "UPIPE_ERR_HIP";
    default: return "UPIPE_ERR_UNKNOWN";
  }
}

int upipe_version(void) { return 100; }

int upipe_gqa_schedule(int H, int Hkv, int C, int U, int* stage_heads,
                       int* kv_stage) {
  if (H < 1 || Hkv < 1 || C < 1 || U < 1 || !stage_heads || !kv_stage)
    return UPIPE_ERR_INVALID_ARG;
  if (H % Hkv || U % C || H % U || H % C || Hkv % C) return UPIPE_ERR_INVALID_ARG;
  const int G = H / Hkv, per_dev = H / C, per_stage = U / C;
  for (int g = 0; g < Hkv; ++g) kv_stage[g] = -1;
  int n = 0;
  for (int s = 0; s < H / U; ++s)
    for (int p = 0; p < C; ++p)
      for (int j = 0; j < per_stage; ++j) {
        const int h = p * per_dev + s * per_stage + j;
        stage_heads[n++] = h;
        if (kv_stage[h / G] < 0) kv_stage[h / G] = s;
      }
  return UPIPE_OK;
}

size_t upipe_attn_fwd_workspace_size(int64_t S, int Hq, int Hkv, int d, int U) {
  if (check_attn_shape(S, Hq, Hkv, d, U) != UPIPE_OK) return 0;
  return plan_attn_fwd(S, Hq, Hkv, U).total;
}

size_t upipe_attn_bwd_workspace_size(int64_t S, int Hq, int Hkv, int d, int U) {
  if (check_attn_shape(S, Hq, Hkv, d, U) != UPIPE_OK) return 0;
  return plan_attn_bwd(S, Hq, Hkv, U).total;
}

static int attn_fwd_batch(const void* q, const void* k, const void* v, void* o, float* lse,
                          int64_t B, int64_t S, int Hq, int Hkv, int d, int causal, int U,
                          void* ws, size_t ws_bytes, hipStream_t stream) {
  try {
    int rc = check_attn_shape(S, Hq, Hkv, d, U);
    if (rc != UPIPE_OK) return rc;
    if (!batch_ok(B, S * Hq * HEAD_DIM)) return UPIPE_ERR_INVALID_ARG;
    if (causal != 0 && causal != 1) return UPIPE_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) ||
        !aligned16(lse) || !aligned16(ws))
      return UPIPE_ERR_INVALID_ARG;
    if (ws_bytes < plan_attn_fwd(S, Hq, Hkv, U).total) return UPIPE_ERR_WORKSPACE;
    return run_attn_fwd((const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, lse, B, S, Hq,
                        Hkv, causal, U, (char*)ws, stream);
  } catch (...) {
    return UPIPE_ERR_HIP;
  }
}

int upipe_attn_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int64_t S,
                   int Hq, int Hkv, int d, int causal, int U, void* ws, size_t ws_bytes,
                   hipStream_t stream) {
  return attn_fwd_batch(q, k, v, o, lse, 1, S, Hq, Hkv, d, causal, U, ws, ws_bytes, stream);
}

int upipe_attn_fwd_batch(const void* q, const void* k, const void* v, void* o, float* lse,
                         int64_t B, int64_t S, int Hq, int Hkv, int d, int causal, int U,
                         void* ws, size_t ws_bytes, hipStream_t stream) {
  return attn_fwd_batch(q, k, v, o, lse, B, S, Hq, Hkv, d, causal, U, ws, ws_bytes, stream);
}

size_t upipe_attn_fwd_ring_workspace_size(int64_t Sq, int64_t Skv, int Hq, int Hkv, int d, int U) {
  if (check_attn_shape(Sq, Hq, Hkv, d, U) != UPIPE_OK) return 0;
  if (check_attn_shape(Skv, Hq, Hkv, d, U) != UPIPE_OK) return 0;
  return plan_attn_fwd_ring(Sq, Skv, Hq, Hkv, U).total;
}

int upipe_attn_fwd_ring(const void* q, const void* k, const void* v, void* o, float* lse,
                        int64_t Sq, int64_t Skv, int64_t q_offset, int64_t kv_offset, int Hq,
                        int Hkv, int d, int causal, int U, void* ws, size_t ws_bytes,
                        hipStream_t stream) {
  try {
    int rc = check_attn_shape(Sq, Hq, Hkv, d, U);
    if (rc != UPIPE_OK) return rc;
    rc = check_attn_shape(Skv, Hq, Hkv, d, U);
    if (rc != UPIPE_OK) return rc;
    if (causal != 0 && causal != 1) return UPIPE_ERR_INVALID_ARG;
    const int64_t lim = int64_t(1) << 62;
    if (q_offset < -lim || q_offset > lim || kv_offset < -lim || kv_offset > lim)
      return UPIPE_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) ||
        !aligned16(lse) || !aligned16(ws))
      return UPIPE_ERR_INVALID_ARG;
    int64_t delta;   // q_offset - kv_offset; fits unless it is exactly 2^63
    if (__builtin_sub_overflow(q_offset, kv_offset, &delta)) return UPIPE_ERR_INVALID_ARG;
    if (ws_bytes < plan_attn_fwd_ring(Sq, Skv, Hq, Hkv, U).total) return UPIPE_ERR_WORKSPACE;
    return run_attn_fwd_ring((const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, lse, 1, Sq,
                             Skv, delta, Hq, Hkv, causal, U, (char*)ws, stream);
  } catch (...) {
    return UPIPE_ERR_HIP;
  }
}

int upipe_lse_merge(void* o, float* lse, const void* o_part, const float* lse_part, int64_t S,
                    int H, int d, hipStream_t stream) {
  try {
    if (S < 1 || H < 1) return UPIPE_ERR_INVALID_ARG;
    if (d != HEAD_DIM) return UPIPE_ERR_UNSUPPORTED;
    if (H > kMaxHeads || S > kMaxSeq) return UPIPE_ERR_UNSUPPORTED;
    if (!aligned16(o) || !aligned16(lse) || !aligned16(o_part) || !aligned16(lse_part))
      return UPIPE_ERR_INVALID_ARG;
    UPIPE_LAUNCH(kLseMerge, stream,
                 launch_lse_merge((bf16*)o, lse, (const bf16*)o_part, lse_part, S, H, stream));
    return UPIPE_OK;
  } catch (...) {
    return UPIPE_ERR_HIP;
  }
}

int upipe_rope(void* x, int64_t S, int H, int d, int64_t pos0, double base, int inverse,
               hipStream_t stream) {
  try {
    if (S < 0 || H < 1 || (inverse != 0 && inverse != 1) || base == 0.0)
      return UPIPE_ERR_INVALID_ARG;
    if (d != HEAD_DIM) return UPIPE_ERR_UNSUPPORTED;
    if (H > kMaxHeads || S > kMaxSeq) return UPIPE_ERR_UNSUPPORTED;
    RopeArgs r;
    const int rc = make_rope(base, pos0, S, &r);
    if (rc != UPIPE_OK) return rc;
    if (!aligned16(x)) return UPIPE_ERR_INVALID_ARG;
    if (S == 0) return UPIPE_OK;
    UPIPE_LAUNCH(kRope, stream,
                 launch_rope((bf16*)x, S, H, (int64_t)H * HEAD_DIM, HEAD_DIM, r, inverse, stream));
    return UPIPE_OK;
  } catch (...) {
    return UPIPE_ERR_HIP;
  }
}

static int attn_bwd_batch(const void* q, const void* k, const void* v, const void* o,
                          const float* lse, const void* dout, void* dq, void* dk, void* dv,
                          int64_t B, int64_t S, int Hq, int Hkv, int d, int causal, int U,
                          void* ws, size_t ws_bytes, hipStream_t stream) {
  try {
    int rc = check_attn_shape(S, Hq, Hkv, d, U);
    if (rc != UPIPE_OK) return rc;
    if (!batch_ok(B, S * Hq * HEAD_DIM)) return UPIPE_ERR_INVALID_ARG;
    if (causal != 0 && causal != 1) return UPIPE_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) ||
        !aligned16(lse) || !aligned16(dout) || !aligned16(dq) || !aligned16(dk) ||
        !aligned16(dv) || !aligned16(ws))
      return UPIPE_ERR_INVALID_ARG;
    if (ws_bytes < plan_attn_bwd(S, Hq, Hkv, U).total) return UPIPE_ERR_WORKSPACE;
    return run_attn_bwd((const bf16*)q, (const bf16*)k, (const bf16*)v, (const bf16*)o, lse,
                        (const bf16*)dout, (bf16*)dq, (bf16*)dk, (bf16*)dv, B, S, Hq, Hkv, causal,
                        U, (char*)ws, stream);
  } catch (...) {
    return UPIPE_ERR_HIP;
  }
}

int upipe_attn_bwd(const void* q, const void* k, const void* v, const void* o, const float* lse,
                   const void* dout, void* dq, void* dk, void* dv, int64_t S, int Hq, int Hkv,
                   int d, int causal, int U, void* ws, size_t ws_bytes, hipStream_t stream) {
  return attn_bwd_batch(q, k, v, o, lse, dout, dq, dk, dv, 1, S, Hq, Hkv, d, causal, U, ws,
                        ws_bytes, stream);
}

int upipe_attn_bwd_batch(const void* q, const void* k, const void* v, const void* o,
                         const float* lse, const void* dout, void* dq, void* dk, void* dv,
                         int64_t B, int64_t S, int Hq, int Hkv, int d, int causal, int U,
                         void* ws, size_t ws_bytes, hipStream_t stream) {
  return attn_bwd_batch(q, k, v, o, lse, dout, dq, dk, dv, B, S, Hq, Hkv, d, causal, U, ws,
                        ws_bytes, stream);
}

int upipe_profile_enable(int on) {
  prof().on = on != 0;
  return UPIPE_OK;
}

int upipe_profile_reset(void) {
  Profiler& p = prof();
  for (auto& r : p.recs) {
    p.pool.push_back(r.start);
    p.pool.push_back(r.stop);
  }
  p.recs.clear();
  return UPIPE_OK;
}

int upipe_profile_query(const char* name, int* launches, double* total_ms) {
  if (!name || !launches || !total_ms) return UPIPE_ERR_INVALID_ARG;
  int fam = -1;
  for (int i = 0; i < kNumFamilies; ++i)
    if (strcmp(name, kFamilyNames[i]) == 0) fam = i;
  if (fam < 0) return UPIPE_ERR_INVALID_ARG;
  int n = 0;
  double ms = 0.0;
  for (auto& r : prof().recs) {
    if (r.family != fam) continue;
    if (hipEventSynchronize(r.stop) != hipSuccess) return UPIPE_ERR_HIP;
    float e = 0.f;
    if (hipEventElapsedTime(&e, r.start, r.stop) != hipSuccess) return UPIPE_ERR_HIP;
    ms += e;
    ++n;
  }
  *launches = n;
  *total_ms = ms;
  return UPIPE_OK;
}

const char* upipe_profile_name(int i) {
  return (i >= 0 && i < kNumFamilies) ? kFamilyNames[i] : nullptr;
}

}  // extern "C"
