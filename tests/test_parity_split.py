"""GPU parity where a launch rule changes.

Forward: a stage's keys are split into 1, 2 or 4 parts by the number of 256-row
query blocks times heads, and keys and values are packed only when one head's
token-major rows span 2^32 bytes; up to 128 queries take more than 8192 keys in
two halves.  Query counts end one row into a block, on it and before it; the key
ranges are short, so the oracle stays cheap.

Backward: dK/dV cuts the walk over a key block's query tiles into segments,
with 128 or 64 keys a workgroup, and dQ splits keys like the forward; tensors
that overlap an output take the path that packs them (test_parity_overlap.py), and
so do long ones (test_parity_long.py).

Products: 256 x 256 or 128 x 128 tiles by how they fill the chip."""

import numpy as np
import pytest
import torch

import workloads as W
from oracle import attention as A
from oracle import layer as L
from oracle import ring as R
from tol import as64, assert_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _upipe():
    from paper_2602_21196_amd import upipe
    upipe.lib()
    return upipe


def _bits(t):
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32)


def _qkv(Sq, Skv, Hq, Hkv, seed):
    g = torch.Generator().manual_seed(seed)
    return tuple(torch.randn(s, generator=g).to(torch.bfloat16)
                 for s in ((Sq, Hq, 128), (Skv, Hkv, 128), (Skv, Hkv, 128)))


# Sq, Skv, Hq, Hkv, offset of the queries, causal: 256-row blocks x heads on both
# sides of 64 | 128 (every key visible) and 224 | 448 (causal).
PARTS = [
    (16384, 130, 1, 1, 0, False), (16385, 130, 1, 1, 0, False),    # 64 | 65
    (8192, 300, 4, 2, 300, True), (8193, 300, 4, 2, 300, True),    # 128 | 132, all visible
    (7168, 257, 8, 2, -7000, True), (7169, 257, 8, 2, -7000, True),    # 224 | 232
    (14336, 100, 8, 1, 50, True), (14337, 100, 8, 1, -14300, True),    # 448 | 456
    (33, 127, 2, 1, 90, True), (65, 129, 2, 2, 64, True), (127, 33, 1, 1, 0, False),
]


@pytest.mark.parametrize("Sq,Skv,Hq,Hkv,off,causal", PARTS)
def test_forward_key_parts(Sq, Skv, Hq, Hkv, off, causal):
    """Bars: tol.py's, for bf16 o and fp32 lse."""
    up = _upipe()
    q, k, v = _qkv(Sq, Skv, Hq, Hkv, Sq + Skv)
    rows = np.unique(np.r_[0:min(Sq, 70), max(0, Sq - 300):Sq,
                           np.random.default_rng(Sq).integers(0, Sq, 200)])
    print(f"key parts Sq={Sq} Skv={Skv} Hq={Hq} off={off} causal={causal}", flush=True)
    o, lse = up.attn_fwd_ring(q.to(DEV), k.to(DEV), v.to(DEV), off, 0, causal=causal, U=1)
    torch.cuda.synchronize()
    o, lse = o.cpu()[rows], lse.cpu()[:, rows].double().numpy()
    o_ref, lse_ref = R.attn_fwd_offset(as64(q), as64(k), as64(v), off, causal)
    o_ref, lse_ref = o_ref[rows], lse_ref[:, rows]
    assert_close("o", o, o_ref)
    empty = np.isneginf(lse_ref)
    assert np.array_equal(np.isneginf(lse), empty)
    assert np.all(o.float().numpy()[empty.T] == 0)
    assert_close("lse", torch.from_numpy(np.where(empty, 0.0, lse)), np.where(empty, 0.0, lse_ref))


def test_forward_packs_keys_beyond_32_bit_offsets():
    """2^20 keys of 16 heads: one head's rows span 2^32 bytes, so they are
    packed; each head is bitwise what it is alone, where its rows are read in
    place."""
    up = _upipe()
    Sq, Skv, H = 40, 1 << 20, 16
    g = torch.Generator(device=DEV).manual_seed(5)
    q = torch.randn((Sq, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    k = torch.randn((Skv, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn((Skv, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    o, lse = up.attn_fwd_ring(q, k, v, Skv, 0, causal=True, U=4)
    for h in (0, 7, 15):
        o1, l1 = up.attn_fwd_ring(q[:, h:h + 1].contiguous(), k[:, h:h + 1].contiguous(),
                                  v[:, h:h + 1].contiguous(), Skv, 0, causal=True, U=1)
        torch.cuda.synchronize()
        assert torch.equal(_bits(o[:, h]), _bits(o1[:, 0])), h
        assert torch.equal(_bits(lse[h]), _bits(l1[0])), h


# One to 16 query tiles, one group and several, odd groups, remainders of
# segments and tiles; the workspace bounds the segments, and it is smallest at
# different chunk sizes (with and without carries).
BACKWARD = [(129, 3, 1, True), (385, 3, 3, True), (640, 5, 1, True), (897, 16, 4, True),
            (1409, 6, 1, True), (2049, 1, 1, True), (2047, 12, 2, True), (1281, 7, 1, False),
            (1152, 4, 4, False), (1920, 16, 2, False)]


@pytest.mark.parametrize("S,Hq,Hkv,causal", BACKWARD)
def test_backward_segments(S, Hq, Hkv, causal):
    """Against the oracle (tol.py's bars) and bitwise equal for every U."""
    up = _upipe()
    cpu = W.attention_inputs(S, Hq, Hkv, 128, 40 + S)
    ref = A.attn_bwd(*(as64(t) for t in cpu), causal)
    q, k, v, do = (t.to(DEV) for t in cpu)
    first = None
    for U in [u for u in range(1, Hq + 1) if Hq % u == 0]:
        print(f"segments S={S} Hq={Hq} Hkv={Hkv} causal={causal} U={U}", flush=True)
        o, lse = up.attn_fwd(q, k, v, causal=causal, U=U)
        got = up.attn_bwd(q, k, v, o, lse, do, causal=causal, U=U)
        torch.cuda.synchronize()
        if first is None:
            first = got
            for name, a, r in zip(("dq", "dk", "dv"), got, ref):
                assert_close(name, a.cpu(), r)
        for a, b in zip(first, got):
            assert torch.equal(_bits(a), _bits(b)), U


# 256-row blocks x heads on both sides of 224 | 448 (causal) and 64 | 128.
DQ_PARTS = [(3584, 16, 2, True), (3585, 16, 2, True), (7169, 16, 4, True), (1025, 14, 2, False),
            (2305, 14, 7, False)]


@pytest.mark.parametrize("S,Hq,Hkv,causal", DQ_PARTS)
def test_dq_key_parts(S, Hq, Hkv, causal):
    """dQ rows at both ends of the sequence, of 32-row waves and at random; bars: tol.py's."""
    up = _upipe()
    cpu = W.attention_inputs(S, Hq, Hkv, 128, 60 + S)
    rows = np.unique(np.r_[0:34, 223:258, S - 66:S, np.random.default_rng(S).integers(0, S, 60)])
    q, k, v, do = (t.to(DEV) for t in cpu)
    print(f"dq parts S={S} Hq={Hq} Hkv={Hkv} causal={causal}", flush=True)
    o, lse = up.attn_fwd(q, k, v, causal=causal, U=2)
    dq, _, _ = up.attn_bwd(q, k, v, o, lse, do, causal=causal, U=2)
    torch.cuda.synchronize()
    q, k, v, do = cpu
    _, _, ref, _ = A.attn_rows_at(as64(q[rows]), rows, as64(k), as64(v), as64(do[rows]), causal)
    assert_close("dq", dq.cpu()[rows], ref)


def test_backward_of_a_long_batch_equals_single_sequences():
    """More sequences than rows are kept for at a time."""
    up = _upipe()
    q, k, v, do = (t.to(DEV) for t in W.batch_attention_inputs(600, 4, 2, 128, 77, 6))
    o, lse = up.attn_fwd(q, k, v, U=2)
    got = up.attn_bwd(q, k, v, o, lse, do, U=2)
    for b in range(6):
        one = up.attn_bwd(q[b], k[b], v[b], o[b], lse[b], do[b], U=2)
        torch.cuda.synchronize()
        for x, y in zip(got, one):
            assert torch.equal(_bits(x[b]), _bits(y)), b


@pytest.mark.parametrize("over", ["dout", "q"])
def test_backward_gradient_over_an_input(over):
    """dq in the place of dout or q: those are read before they are written."""
    up = _upipe()
    S, Hq, Hkv = 700, 4, 1
    cpu = W.attention_inputs(S, Hq, Hkv, 128, 9)
    ref = A.attn_bwd(*(as64(t) for t in cpu), True)
    q, k, v, do = (t.to(DEV) for t in cpu)
    o, lse = up.attn_fwd(q, k, v, U=1)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    dq = do if over == "dout" else q
    ws = up.workspace(up.upipe_attn_bwd_workspace_size(S, Hq, Hkv, 128, 1), DEV)
    st = up.upipe_attn_bwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(),
                           do.data_ptr(), dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), S, Hq, Hkv,
                           128, 1, 1, ws.data_ptr(), ws.numel(),
                           torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    for name, a, r in zip(("dq", "dk", "dv"), (dq, dk, dv), ref):
        assert_close(name, a.cpu(), r)


@pytest.mark.parametrize("M,N,K", [(8320, 4224, 128), (8192, 4096, 384), (16512, 640, 256)])
def test_product_with_large_tiles(M, N, K):
    """Half tiles at both edges; against the float64 product (entries grow like
    sqrt(K): the bar on the rms-scaled error), and bitwise what the first rows
    alone give, which take the small tiles."""
    up = _upipe()
    g = torch.Generator().manual_seed(M + K)
    a = torch.randn((M, K), generator=g).to(torch.bfloat16)
    b = torch.randn((K, N), generator=g).to(torch.bfloat16)
    c = up.gemm(a.to(DEV), b.to(DEV))
    few = up.gemm(a[:640].to(DEV), b.to(DEV))
    torch.cuda.synchronize()
    assert torch.equal(_bits(c[:640]), _bits(few))
    assert_close("c", c.cpu(), as64(a) @ as64(b), rms_scaled=True)


def test_block_projection_with_large_tiles():
    """16300 rows of 3 + 2 heads: a ragged M and half a tile along N.  The block is
    causal, so its first rows are those of the sequence's beginning (oracle)."""
    up = _upipe()
    S, dm, Hq, Hkv, n = 16300, 256, 3, 1, 700
    x, wqkv, wo, _ = W.layer_inputs(S, dm, Hq, Hkv, 128, 21, w_std=0.06)
    y, o, lse = up.layer_fwd(x.to(DEV), wqkv.to(DEV), wo.to(DEV), Hq, Hkv, U=1, rope_base=1e4)
    torch.cuda.synchronize()
    y_r, o_r, lse_r = L.layer_fwd(as64(x[:n]), as64(wqkv), as64(wo), Hq, Hkv, 128, rope_base=1e4)
    assert_close("y", y[:n].cpu(), y_r)
    assert_close("o", o[:n].cpu(), o_r)
    assert_close("lse", lse[:, :n].cpu(), lse_r)


@pytest.mark.parametrize("S,dm,Hq,Hkv,B", [(150, 256, 40, 1, 1), (129, 128, 40, 8, 2),
                                           (700, 128, 64, 64, 1)])
def test_block_recomputes_many_heads_in_little_room(S, dm, Hq, Hkv, B):
    """At U = 1 and 40 heads or more the workspace has no room of its own for the
    recomputed attention output: it lies in the dK | dV part of dQKV, twice the
    key/value heads at a time.  Gradients are bitwise those with the output kept,
    and a workspace of the size query's bytes is enough."""
    up = _upipe()
    x, wqkv, wo, dy = (t.to(DEV) for t in W.batch_layer_inputs(S, dm, Hq, Hkv, 128, 8, B))
    size = up.upipe_layer_bwd_workspace_size(S, dm, Hq, Hkv, 128, 1)
    guard = 4096
    ws = torch.full((size + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    print(f"recompute S={S} dm={dm} Hq={Hq} Hkv={Hkv} B={B}", flush=True)
    _, o, lse = up.layer_fwd(x, wqkv, wo, Hq, Hkv, U=1, rope_base=1e4)
    kept = up.layer_bwd(x, wqkv, wo, o, lse, dy, Hq, Hkv, U=1, rope_base=1e4)
    full = up.layer_bwd(x, wqkv, wo, None, None, dy, Hq, Hkv, U=1, rope_base=1e4, ws=ws)
    torch.cuda.synchronize()
    for a, b in zip(kept, full):
        assert torch.equal(_bits(a), _bits(b))
    assert bool((ws[size:] == 0xA5).all())


# 64-key workgroups (few key blocks), 128-key ones in segments (8 x 32 key blocks),
# and the walk of a key block by one workgroup (dq over dout).
@pytest.mark.parametrize("S,Hq,Hkv,over", [(512, 2, 1, False), (4096, 8, 8, False),
                                           (1000, 4, 2, True), (384, 2, 2, True)])
@pytest.mark.parametrize("where,value", [("q", float("nan")), ("q", float("inf")),
                                         ("dout", float("nan")), ("dout", -float("inf"))])
def test_nonfinite_rows_stay_in_their_half_tile(S, Hq, Hkv, over, where, value):
    """A query row that holds an infinity or NaN changes dk and dv only of keys it sees
    or shares a half tile (64 rows) with; later keys keep every bit."""
    up = _upipe()
    q, k, v, do = (t.to(DEV) for t in W.attention_inputs(S, Hq, Hkv, 128, 17))
    o, lse = up.attn_fwd(q, k, v, U=1)
    ws = up.workspace(up.upipe_attn_bwd_workspace_size(S, Hq, Hkv, 128, 1), DEV)

    def bwd(q, do):
        dk, dv = torch.empty_like(k), torch.empty_like(v)
        do = do.clone()
        dq = do if over else torch.empty_like(q)
        st = up.upipe_attn_bwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(),
                               lse.data_ptr(), do.data_ptr(), dq.data_ptr(), dk.data_ptr(),
                               dv.data_ptr(), S, Hq, Hkv, 128, 1, 1, ws.data_ptr(), ws.numel(),
                               torch.cuda.current_stream().cuda_stream)
        assert st == 0
        torch.cuda.synchronize()
        return dk, dv

    clean = bwd(q, do)
    for r in (0, 10, 63, 64, 127, 130, 191, 192, 255, S - 65):
        print(f"nonfinite S={S} Hq={Hq} over={over} {where} row {r} {value}", flush=True)
        x = {"q": q.clone(), "dout": do.clone()}
        x[where][r, Hq - 1, 5] = value
        got = bwd(x["q"], x["dout"])
        first = (r // 64 + 1) * 64
        # (with q infinite a score may be -inf: p = 0, and dv does not change)
        assert not all(bool(torch.isfinite(b[:r + 1].float()).all()) for b in got)
        for a, b in zip(clean, got):
            assert torch.equal(_bits(a[first:]), _bits(b[first:])), r


# Sq, Skv, Hq, Hkv, offset of the queries, causal: up to 128 queries and more than
# 8192 visible keys take the keys in two halves.  One key/value head of a length
# that is a multiple of 128 leaves little workspace: with few heads a chunk the
# halves run one after the other, with all of them (and with packed keys' room)
# side by side.  The last rows end where the second half begins, or see no key.
HALVES = [(1, 8193, 1, 1, 8192, True), (128, 8320, 4, 1, 8320, True), (33, 8448, 8, 2, 9000, True),
          (64, 9000, 4, 4, 8200, True), (65, 16384, 2, 1, 8150, True), (128, 8300, 2, 1, 0, False),
          (100, 8321, 64, 1, 8321, True), (128, 8192, 2, 1, 8192, True),
          (127, 12288, 2, 1, 8064, True), (128, 30000, 2, 1, -60, True)]


@pytest.mark.parametrize("Sq,Skv,Hq,Hkv,off,causal", HALVES)
def test_forward_key_halves(Sq, Skv, Hq, Hkv, off, causal):
    """Against the oracle (tol.py's bars), bitwise equal for every U and with o in the
    place of q, which always takes the halves one after the other."""
    up = _upipe()
    q, k, v = _qkv(Sq, Skv, Hq, Hkv, Sq + Skv)
    o_ref, lse_ref = R.attn_fwd_offset(as64(q), as64(k), as64(v), off, causal)
    empty = np.isneginf(lse_ref)
    q, k, v = (t.to(DEV) for t in (q, k, v))
    first = None
    for U in [u for u in range(1, Hq + 1) if Hq % u == 0]:
        print(f"key halves Sq={Sq} Skv={Skv} Hq={Hq} Hkv={Hkv} off={off} U={U}", flush=True)
        ws = up.workspace(up.upipe_attn_fwd_ring_workspace_size(Sq, Skv, Hq, Hkv, 128, U), DEV)
        ws.fill_(0xFF)
        o, lse = up.attn_fwd_ring(q, k, v, off, 0, causal=causal, U=U, ws=ws)
        qo, lse2 = q.clone(), torch.empty_like(lse)
        assert up.upipe_attn_fwd_ring(qo.data_ptr(), k.data_ptr(), v.data_ptr(), qo.data_ptr(),
                                      lse2.data_ptr(), Sq, Skv, off, 0, Hq, Hkv, 128, int(causal),
                                      U, ws.data_ptr(), ws.numel(),
                                      torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        if first is None:
            first = (o, lse)
            lse_np = lse.cpu().double().numpy()
            assert_close("o", o.cpu(), o_ref)
            assert np.array_equal(np.isneginf(lse_np), empty)
            assert_close("lse", torch.from_numpy(np.where(empty, 0.0, lse_np)),
                         np.where(empty, 0.0, lse_ref))
        for a, b, c in zip(first, (o, lse), (qo, lse2)):
            assert torch.equal(_bits(a), _bits(b)) and torch.equal(_bits(a), _bits(c)), U
