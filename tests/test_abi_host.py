"""The C ABI on the host: it loads, exports what the header declares, and
validates arguments before any GPU work (no kernel is launched here)."""

import ctypes
import os
import re

import pytest

from oracle import schedule as SCH
from paper_2602_21196_amd import upipe

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "upipe.h")


def _declared():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(upipe_[a-z0-9_]+)\s*\(", src)))


def test_library_loads_and_exports_every_declared_symbol():
    lib = upipe.lib()
    names = _declared()
    assert len(names) >= 15
    for n in names:
        assert hasattr(lib, n), f"{n} declared in upipe.h but not exported"
        assert n in upipe._SIGNATURES, f"{n} has no Python mirror"


def test_status_strings_and_version():
    assert upipe.upipe_status_string(0) == "UPIPE_OK"
    assert upipe.upipe_status_string(-3) == "UPIPE_ERR_WORKSPACE"
    assert upipe.upipe_status_string(7) == "UPIPE_ERR_UNKNOWN"
    assert upipe.upipe_version() >= 100
    assert "attn_fwd" in upipe.upipe_profile_names()


FAKE = 1 << 20   # a 16-byte aligned non-null address; never dereferenced


def _call(plain, batch, a, kw):
    """The contract call without B; with B in kw, only the batched call.
    Without B both run and must agree (B = 1 is the contract call)."""
    a.update(kw)
    if "B" in kw:
        return batch(*a.values())
    b = a.pop("B")
    r = plain(*a.values())
    a["B"] = b
    order = list(a)   # B sits before S in the batched signature
    args = [a[n] for n in order[:order.index("S")] if n != "B"] + [1] + \
        [a[n] for n in order[order.index("S"):] if n != "B"]
    assert batch(*args) == r
    return r


def _fwd(**kw):
    a = dict(q=FAKE, k=FAKE, v=FAKE, o=FAKE, lse=FAKE, B=1, S=512, Hq=4, Hkv=1,
             d=128, causal=1, U=1, ws=FAKE, ws_bytes=1 << 40, stream=None)
    return _call(upipe.upipe_attn_fwd, upipe.upipe_attn_fwd_batch, a, kw)


def _bwd(**kw):
    a = dict(q=FAKE, k=FAKE, v=FAKE, o=FAKE, lse=FAKE, dout=FAKE, dq=FAKE,
             dk=FAKE, dv=FAKE, B=1, S=512, Hq=4, Hkv=1, d=128, causal=1, U=1,
             ws=FAKE, ws_bytes=1 << 40, stream=None)
    return _call(upipe.upipe_attn_bwd, upipe.upipe_attn_bwd_batch, a, kw)


# The four compute calls of the boundary, parameter by parameter.
CONTRACT = {
    "upipe_attn_fwd": ["const void*"] * 3 + ["void*", "float*", "int64_t"] + ["int"] * 5 +
                      ["void*", "size_t", "hipStream_t"],
    "upipe_attn_bwd": ["const void*"] * 4 + ["const float*", "const void*"] + ["void*"] * 3 +
                      ["int64_t"] + ["int"] * 5 + ["void*", "size_t", "hipStream_t"],
    "upipe_layer_fwd": ["const void*"] * 3 + ["void*", "void*", "float*", "int64_t"] +
                       ["int"] * 5 + ["void*", "size_t", "hipStream_t"],
    "upipe_layer_bwd": ["const void*"] * 4 + ["const float*", "const void*"] + ["void*"] * 3 +
                       ["int64_t"] + ["int"] * 5 + ["void*", "size_t", "hipStream_t"],
}
_CTYPE = {"const void*": ctypes.c_void_p, "void*": ctypes.c_void_p,
          "float*": ctypes.c_void_p, "const float*": ctypes.c_void_p,
          "int64_t": ctypes.c_int64, "int": ctypes.c_int, "size_t": ctypes.c_size_t,
          "hipStream_t": ctypes.c_void_p}


def _prototype(name):
    src = re.sub(r"/\*.*?\*/", "", open(HEADER).read(), flags=re.S)
    m = re.search(r"\bint\s+" + name + r"\s*\(([^)]*)\)", src)
    assert m, name
    types = []
    for par in m.group(1).split(","):
        par = " ".join(par.split())
        par = re.sub(r"\s*\*\s*", "* ", par).strip()
        types.append(par.rsplit(" ", 1)[0].replace("* ", "*").strip())
    return types


@pytest.mark.parametrize("name", sorted(CONTRACT))
def test_contract_signatures(name):
    """upipe_attn_fwd / upipe_attn_bwd / upipe_layer_fwd / upipe_layer_bwd take
    exactly the contract's parameters, in the header and in the binding."""
    assert _prototype(name) == CONTRACT[name]
    assert upipe._SIGNATURES[name][1] == [_CTYPE[t] for t in CONTRACT[name]]


@pytest.mark.parametrize("fn", [_fwd, _bwd])
def test_argument_validation(fn):
    INV, UNS, WS = -1, -2, -3
    assert fn(S=0) == INV
    assert fn(Hq=4, Hkv=3) == INV             # Hkv does not divide Hq
    assert fn(U=3) == INV                     # U does not divide Hq
    assert fn(U=0) == INV
    assert fn(d=64) == UNS
    assert fn(Hq=128, Hkv=1, U=1) == UNS
    assert fn(q=None) == INV
    assert fn(q=FAKE + 8) == INV              # misaligned
    assert fn(ws=None) == INV
    assert fn(causal=2) == INV
    assert fn(ws_bytes=1024) == WS
    assert fn(B=0) == INV
    assert fn(B=-1) == INV
    assert fn(B=8, ws_bytes=1024) == WS       # a batch needs no more workspace
    # B times one sequence's [S, Hq, d] must stay below 2^61 elements
    per_seq = 512 * 4 * 128
    assert fn(B=(1 << 61) // per_seq, ws_bytes=1024) == WS
    assert fn(B=(1 << 61) // per_seq + 1, ws_bytes=1024) == INV


def _ring(**kw):
    a = dict(q=FAKE, k=FAKE, v=FAKE, o=FAKE, lse=FAKE, Sq=512, Skv=384, q_offset=1000,
             kv_offset=200, Hq=4, Hkv=1, d=128, causal=1, U=1, ws=FAKE,
             ws_bytes=1 << 40, stream=None)
    a.update(kw)
    return upipe.upipe_attn_fwd_ring(*a.values())


def test_ring_step_validation_and_workspace():
    INV, UNS, WS = -1, -2, -3
    assert _ring(Sq=0) == INV
    assert _ring(Skv=0) == INV
    assert _ring(Hq=4, Hkv=3) == INV
    assert _ring(U=3) == INV
    assert _ring(d=64) == UNS
    assert _ring(causal=2) == INV
    assert _ring(q_offset=(1 << 62) + 1) == INV
    assert _ring(kv_offset=-(1 << 62) - 1) == INV
    # the offset difference must fit in int64: 2^62 - (-2^62) = 2^63 does not
    assert _ring(q_offset=1 << 62, kv_offset=-(1 << 62), ws_bytes=1024) == INV
    assert _ring(q_offset=1 << 62, kv_offset=1 - (1 << 62), ws_bytes=1024) == WS
    assert _ring(q_offset=-(1 << 62), kv_offset=1 << 62, ws_bytes=1024) == WS
    assert _ring(k=None) == INV
    assert _ring(lse=FAKE + 4) == INV
    assert _ring(ws_bytes=1024) == WS
    # The sizes that callers may have saved: K, V packed at the key length; Q, O
    # chunk buffers at the query length.  Few query blocks (at most 128 of 256
    # rows) and at least two key stages: a second O buffer and fp32 lse rows, for
    # the key range in two halves.
    qh, kh = 512 * 128 * 2, 384 * 128 * 2
    # One key/value head and 384 = 3 x 128 keys: K, V are read in place.
    for U in (1, 2, 4):
        assert upipe.upipe_attn_fwd_ring_workspace_size(512, 384, 4, 1, 128, U) == \
            U * qh + 2 * U * qh + 2 * U * 512 * 4
        assert upipe.upipe_attn_fwd_ring_workspace_size(512, 384, 4, 2, 128, U) == \
            2 * 2 * kh + U * qh + 2 * U * qh + 2 * U * 512 * 4
    # a single key stage: no second one
    assert upipe.upipe_attn_fwd_ring_workspace_size(512, 128, 4, 1, 128, 1) == 2 * qh
    # a ragged key length is packed (padded) once
    assert upipe.upipe_attn_fwd_ring_workspace_size(512, 100, 4, 1, 128, 1) == \
        2 * 128 * 256 + 2 * qh
    # equal lengths: the plain forward's workspace
    assert upipe.upipe_attn_fwd_ring_workspace_size(1000, 1000, 4, 2, 128, 2) == \
        upipe.upipe_attn_fwd_workspace_size(1000, 4, 2, 128, 2)
    assert upipe.upipe_attn_fwd_ring_workspace_size(512, 0, 4, 1, 128, 1) == 0


def test_lse_merge_validation():
    INV, UNS = -1, -2
    m = upipe.upipe_lse_merge
    assert m(FAKE, FAKE, FAKE, FAKE, 0, 4, 128, None) == INV
    assert m(FAKE, FAKE, FAKE, FAKE, 16, 0, 128, None) == INV
    assert m(FAKE, FAKE, FAKE, FAKE, 16, 4, 64, None) == UNS
    assert m(None, FAKE, FAKE, FAKE, 16, 4, 128, None) == INV
    assert m(FAKE, FAKE, FAKE + 2, FAKE, 16, 4, 128, None) == INV


def test_workspace_sizes_follow_the_plan():
    S, d = 131072, 128
    Sp = S
    head = Sp * d * 2
    for U in (1, 2, 4):
        # one key/value head, S a multiple of 128: K and V read in place
        fwd = upipe.upipe_attn_fwd_workspace_size(S, 4, 1, d, U)
        assert fwd == 2 * U * head
        bwd = upipe.upipe_attn_bwd_workspace_size(S, 4, 1, d, U)
        carry = 4 * head if U < 4 else 0          # fp32 dK, dV accumulators
        # per chunk head Q, dO, dQ and the fp32 D and lse rows
        assert bwd == carry + 3 * U * head + 2 * U * Sp * 4
        # two key/value heads: K, V packed once and resident
        assert upipe.upipe_attn_fwd_workspace_size(S, 4, 2, d, U) == 4 * head + 2 * U * head
        carry2 = 8 * head if U < 2 else 0
        assert upipe.upipe_attn_bwd_workspace_size(S, 4, 2, d, U) == \
            4 * head + carry2 + 3 * U * head + 2 * U * Sp * 4
    # padding of a ragged length to the 128-row granule (one key stage)
    assert upipe.upipe_attn_fwd_workspace_size(1, 1, 1, d, 1) == 4 * 128 * d * 2
    # 32768 rows = 128 query blocks of 256: room for two halves of the keys; one
    # row more makes 129 blocks: none
    s32 = 32768 * d * 2
    assert upipe.upipe_attn_fwd_workspace_size(32768, 4, 1, d, 1) == \
        s32 + 2 * s32 + 2 * 32768 * 4
    s33 = 32896 * d * 2
    assert upipe.upipe_attn_fwd_workspace_size(32769, 4, 1, d, 1) == 2 * s33 + 2 * s33
    assert upipe.upipe_attn_fwd_workspace_size(0, 1, 1, d, 1) == 0
    assert upipe.upipe_attn_fwd_workspace_size(5, 4, 1, 64, 1) == 0
    # longest supported share: 2^24 - 128 rows (32-bit per-head byte offsets)
    smax = (1 << 24) - 128
    assert upipe.upipe_attn_fwd_workspace_size(smax, 1, 1, d, 1) > 0
    assert upipe.upipe_attn_fwd_workspace_size(smax + 1, 1, 1, d, 1) == 0
    assert upipe.upipe_attn_bwd_workspace_size(smax + 1, 1, 1, d, 1) == 0
    # memory grows linearly in U
    sizes = [upipe.upipe_attn_fwd_workspace_size(S, 8, 1, d, U)
             for U in (1, 2, 4, 8)]
    assert sizes[1] - sizes[0] == (sizes[2] - sizes[1]) // 2 == \
        (sizes[3] - sizes[2]) // 4


def _block_backward_size(S, dm, Hq, Hkv, U):
    """The block backward's workspace: what a plan of one chunk of U heads at a time
    needs, in 256-byte aligned pieces."""
    Sp = (S + 127) // 128 * 128
    head = Sp * 256
    G = Hq // Hkv
    carry = any((g * G) // U != ((g + 1) * G - 1) // U for g in range(Hkv))
    piece = max(256, ((S + 31) // 32 + 255) // 256 * 256)
    widest = (Hq + 2 * Hkv) * 128
    used = 0
    for n in ([Hkv * head] * 2 + [2 * Hkv * head] * (2 if carry else 0) +      # K, V, dK32, dV32
              [U * head, U * Sp * 4, U * Sp * 4, U * head, Hq * S * 4] +       # Q, D, lse, O; lse
              [Hq * head, (Hq + 2 * Hkv) * head] +                             # dFO, dQKV
              [(S + piece - 1) // piece * dm * widest * 4] +                   # split-K partials
              [dm * widest * 4, Hq * 128 * dm * 4]):                           # sums over a batch
        used = (used + 255) // 256 * 256 + n
    return used


def test_block_backward_size_stays():
    """Saved sizes stay valid: many heads, chunks of one, short and long, ragged."""
    shapes = [(100, 2048, 64, 8, 1), (129, 128, 64, 8, 1), (12, 256, 40, 8, 1),
              (7, 4096, 40, 40, 1), ((1 << 24) - 128, 1024, 64, 64, 1)]
    for Hq, Hkv in ((1, 1), (4, 1), (8, 2), (33, 3), (40, 1), (40, 8), (48, 16), (64, 1), (64, 64)):
        for U in (u for u in range(1, Hq + 1) if Hq % u == 0):
            for S in (1, 255, 256, 257, 1000, 8192, 8193, 65537, 3113162):
                shapes += [(S, dm, Hq, Hkv, U) for dm in (128, 1024, 8192)]
    for S, dm, Hq, Hkv, U in shapes:
        assert upipe.upipe_layer_bwd_workspace_size(S, dm, Hq, Hkv, 128, U) == \
            _block_backward_size(S, dm, Hq, Hkv, U), (S, dm, Hq, Hkv, U)


@pytest.mark.parametrize("H,Hkv,C,U", [(16, 4, 4, 4), (32, 8, 8, 8),
                                       (64, 8, 8, 8), (64, 16, 4, 8),
                                       (32, 8, 8, 16), (8, 2, 2, 2)])
def test_gqa_schedule_matches_oracle(H, Hkv, C, U):
    st, heads, kv = upipe.upipe_gqa_schedule(H, Hkv, C, U)
    assert st == 0
    stages, kv_stage = SCH.gqa_schedule(H, Hkv, C, U)
    assert heads == [h for s in stages for h in s]
    assert kv == kv_stage


def test_gqa_schedule_rejects_bad_shapes():
    assert upipe.upipe_gqa_schedule(16, 4, 4, 6)[0] == -1
    assert upipe.upipe_gqa_schedule(16, 4, 3, 3)[0] == -1
    assert upipe.upipe_gqa_schedule(0, 4, 4, 4)[0] == -1


def test_layer_entry_points_validate():
    S, dm = 256, 512
    assert upipe.upipe_layer_fwd_workspace_size(S, 500, 4, 1, 128, 1) == 0
    assert upipe.upipe_layer_fwd_workspace_size(S, dm, 4, 1, 64, 1) == 0
    assert upipe.upipe_layer_fwd(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, S, dm, 4,
                                 1, 128, 3, FAKE, 1 << 40, None) == -1
    assert upipe.upipe_layer_fwd_ex(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, S, dm, 4,
                                    1, 128, 3, 0.0, 0, FAKE, 1 << 40, None) == -1
    assert upipe.upipe_layer_fwd_ex(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 0, S, dm, 4,
                                    1, 128, 1, 0.0, 0, FAKE, 1 << 40, None) == -1   # B = 0
    assert upipe.upipe_layer_fwd(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, S, dm, 4,
                                 1, 128, 1, FAKE, 1024, None) == -3
    assert upipe.upipe_layer_bwd(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, S, dm,
                                 4, 1, 128, 1, FAKE, 1024, None) == -3


def _layer(fn, **kw):
    a = dict(B=1, S=256, dm=512, Hq=4, Hkv=1, d=128, U=1, base=5e5, pos0=0)
    a.update(kw)
    if fn == "fwd":
        return upipe.upipe_layer_fwd_ex(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, a["B"], a["S"],
                                        a["dm"], a["Hq"], a["Hkv"], a["d"], a["U"], a["base"],
                                        a["pos0"], FAKE, 0, None)
    return upipe.upipe_layer_bwd_ex(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE,
                                    a["B"], a["S"], a["dm"], a["Hq"], a["Hkv"], a["d"], a["U"],
                                    a["base"], a["pos0"], FAKE, 0, None)


@pytest.mark.parametrize("fn", ["fwd", "bwd"])
def test_layer_rope_arguments_validate(fn):
    INV, UNS, WS = -1, -2, -3
    assert _layer(fn) == WS                      # valid rotary arguments reach the size check
    assert _layer(fn, base=0.0) == WS            # 0: no rotary embedding
    assert _layer(fn, base=-1.0) == INV
    assert _layer(fn, base=float("nan")) == INV
    assert _layer(fn, base=float("inf")) == INV
    assert _layer(fn, pos0=-1) == UNS
    assert _layer(fn, pos0=(1 << 32) - 256) == WS   # last row at 2^32 - 1
    assert _layer(fn, pos0=(1 << 32) - 255) == UNS
    assert _layer(fn, B=4) == WS                 # a batch: same workspace
    assert _layer(fn, B=0) == INV
    assert _layer(fn, B=-3) == INV
    # B times one sequence's largest tensor ([S, d_model] here) below 2^61
    per_seq = 256 * 512
    assert _layer(fn, B=(1 << 61) // per_seq) == WS
    assert _layer(fn, B=(1 << 61) // per_seq + 1) == INV


def test_layer_bwd_saved_output_both_or_neither():
    INV, WS = -1, -3
    S, dm = 256, 512

    def bwd(o, lse):
        r = upipe.upipe_layer_bwd(FAKE, FAKE, FAKE, o, lse, FAKE, FAKE, FAKE, FAKE, S, dm,
                                  4, 1, 128, 1, FAKE, 0, None)
        assert upipe.upipe_layer_bwd_ex(FAKE, FAKE, FAKE, o, lse, FAKE, FAKE, FAKE, FAKE, 1, S,
                                        dm, 4, 1, 128, 1, 0.0, 0, FAKE, 0, None) == r
        return r
    assert bwd(FAKE, FAKE) == WS           # kept output (selective checkpointing)
    assert bwd(None, None) == WS           # recomputed (full checkpointing)
    assert bwd(FAKE, None) == INV
    assert bwd(None, FAKE) == INV
    assert bwd(FAKE + 8, FAKE) == INV      # misaligned


def test_rope_entry_point_validates():
    INV, UNS = -1, -2
    r = upipe.upipe_rope
    assert r(FAKE, 0, 4, 128, 0, 1e4, 0, None) == 0          # empty: nothing to do
    assert r(FAKE, 16, 4, 64, 0, 1e4, 0, None) == UNS
    assert r(FAKE, 16, 0, 128, 0, 1e4, 0, None) == INV
    assert r(FAKE, -1, 4, 128, 0, 1e4, 0, None) == INV
    assert r(FAKE, 16, 4, 128, 0, 0.0, 0, None) == INV       # no "off" for the standalone call
    assert r(FAKE, 16, 4, 128, 0, -2.0, 0, None) == INV
    assert r(FAKE, 16, 4, 128, 0, 1e4, 2, None) == INV
    assert r(FAKE + 8, 16, 4, 128, 0, 1e4, 0, None) == INV   # misaligned
    assert r(FAKE, 16, 4, 128, -5, 1e4, 0, None) == UNS
    assert r(FAKE, 16, 4, 128, (1 << 32) - 15, 1e4, 0, None) == UNS
    assert r(FAKE, 16, 65, 128, 0, 1e4, 0, None) == UNS


def _cpu(*shape):
    import torch
    return torch.zeros(shape, dtype=torch.bfloat16)


def test_torch_wrappers_check_every_shape():
    """The binding checks each tensor's full shape before the library sees a
    raw pointer (a mismatch would be read or written out of bounds on the
    GPU); these CPU tensors never reach a device."""
    import torch
    S, Hq, Hkv, d = 256, 4, 1, 128
    q, k = _cpu(S, Hq, d), _cpu(S, Hkv, d)
    lse = torch.zeros((Hq, S))
    bad = [
        lambda: upipe.attn_fwd(q, _cpu(S, Hkv, 64), k),
        lambda: upipe.attn_fwd(q, k, _cpu(S + 1, Hkv, d)),
        lambda: upipe.attn_fwd(q, _cpu(1, S, Hkv, d), k),
        lambda: upipe.attn_fwd(_cpu(2, S, Hq, d), _cpu(2, S, Hkv, d), _cpu(1, S, Hkv, d)),
        lambda: upipe.attn_bwd(q, k, k, _cpu(S, Hq - 1, d), lse, q),
        lambda: upipe.attn_bwd(q, k, k, q, torch.zeros((Hq, S - 1)), q),
        lambda: upipe.attn_bwd(q, k, k, q, lse, _cpu(S, Hq, d + 8)),
        lambda: upipe.attn_fwd_ring(q, k, _cpu(S, 2, d), 0, 0),
        lambda: upipe.lse_merge(q, lse, _cpu(S, Hq, d), torch.zeros((Hq, S + 1))),
        lambda: upipe.rope(_cpu(S, d), 1e4),
    ]
    dm = 512
    x, wqkv, wo = _cpu(S, dm), _cpu(dm, (Hq + 2 * Hkv) * d), _cpu(Hq * d, dm)
    bad += [
        lambda: upipe.layer_fwd(x, _cpu(dm, (Hq + 1) * d), wo, Hq, Hkv),
        lambda: upipe.layer_fwd(x, wqkv, _cpu(Hq * d, dm + 128), Hq, Hkv),
        lambda: upipe.layer_fwd(x, wqkv, wo, Hq, 2),
        lambda: upipe.layer_bwd(x, wqkv, wo, _cpu(S, Hq, d), lse, _cpu(S, dm - 1), Hq, Hkv),
        lambda: upipe.layer_bwd(x, wqkv, wo, _cpu(S, Hq, 64), lse, x, Hq, Hkv),
        lambda: upipe.layer_bwd(x, wqkv, wo, _cpu(S, Hq, d), torch.zeros((Hq + 1, S)), x,
                                Hq, Hkv),
    ]
    for i, call in enumerate(bad):
        with pytest.raises(ValueError, match="shape|must be|lse_merge"):
            call()
    # right shapes get as far as the device check
    with pytest.raises(ValueError, match="GPU"):
        upipe.attn_fwd(q, k, k)
    with pytest.raises(ValueError, match="GPU"):
        upipe.layer_bwd(x, wqkv, wo, _cpu(S, Hq, d), lse, x, Hq, Hkv)


def test_gemm_entry_point_validates():
    INV, UNS = -1, -2
    g = upipe.upipe_gemm_bf16
    assert g(FAKE, FAKE, FAKE, 0, 128, 128, None) == INV
    assert g(FAKE, FAKE, FAKE, 128, 128, -128, None) == INV
    assert g(FAKE, FAKE, FAKE, 100, 128, 128, None) == UNS
    assert g(FAKE, FAKE, FAKE, 128, 128, 200, None) == UNS
    assert g(FAKE, FAKE, FAKE, 128, 65536 + 128, 128, None) == UNS
    assert g(None, FAKE, FAKE, 128, 128, 128, None) == INV
    assert g(FAKE, FAKE, FAKE + 2, 128, 128, 128, None) == INV
    import torch
    with pytest.raises(ValueError, match="gemm"):
        upipe.gemm(_cpu(128, 256), _cpu(128, 128))
