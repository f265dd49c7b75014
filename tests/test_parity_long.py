"""GPU parity of the attention backward from 65536 rows on: dK/dV head by head on
packed chunks with carried sums, dQ in place for all heads after the last chunk
or, where the rows' terms of all heads do not fit (Hq > 33 U), for each chunk.
Ragged lengths, several key/value heads (strided keys, carries of each head),
every key visible, batches, and keys packed because their rows span 2^32 bytes.
The oracle checks sampled query rows, and key columns conditioned on the GPU's
lse and o; tensors are drawn on the GPU."""

import numpy as np
import pytest
import torch

from oracle import attention as A
from tol import as64, assert_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _upipe():
    from paper_2602_21196_amd import upipe
    upipe.lib()
    return upipe


def _bits(t):
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32)


def _draw(g, *shape):
    """bf16 N(0, 1) on the GPU, in row blocks (no large fp32 temporary)."""
    t = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    flat = t.view(-1)
    for i in range(0, flat.numel(), 1 << 28):
        n = min(1 << 28, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device=DEV)
    return t


def _qkvd(B, S, Hq, Hkv, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return (_draw(g, B, S, Hq, 128), _draw(g, B, S, Hkv, 128), _draw(g, B, S, Hkv, 128),
            _draw(g, B, S, Hq, 128))


def _check(q, k, v, do, o, lse, dq, dk, dv, causal, seed):
    """One sequence, of a few heads."""
    S = q.shape[0]
    rng = np.random.default_rng(seed)
    rows = np.unique(np.r_[0, 127, 128, S - 1, rng.integers(0, S, 12)])
    cols = np.unique(np.r_[0, 127, 128, S - 1, rng.integers(0, S, 6)])
    k64, v64 = as64(k), as64(v)
    o_r, lse_r, dq_r, _ = A.attn_rows_at(as64(q[rows]), rows, k64, v64, as64(do[rows]), causal)
    assert_close("o rows", o[rows].cpu(), o_r)
    assert_close("lse rows", lse[:, rows].cpu(), lse_r)
    assert_close("dq rows", dq[rows].cpu(), dq_r)
    dk_c, dv_c = A.attn_key_cols_given(q.float().cpu().numpy(), do.float().cpu().numpy(), k64, v64,
                                       o.float().cpu().numpy(), lse.cpu().numpy(), cols, causal)
    assert_close("dk cols", dk[cols].cpu(), dk_c)
    assert_close("dv cols", dv[cols].cpu(), dv_c)


# S, Hq, Hkv, B, causal: groups of 2, of 3 that chunks split, and of 1
LONG = [(65537, 4, 2, 1, True), (65537, 4, 2, 2, False), (65664, 6, 2, 1, True),
        (66000, 2, 2, 1, False), (65536, 3, 1, 1, True)]


@pytest.mark.parametrize("S,Hq,Hkv,B,causal", LONG)
def test_long_backward(S, Hq, Hkv, B, causal):
    up = _upipe()
    q, k, v, do = _qkvd(B, S, Hq, Hkv, S + Hq)
    first = None
    for U in [u for u in range(1, Hq + 1) if Hq % u == 0]:
        print(f"long S={S} Hq={Hq} Hkv={Hkv} B={B} causal={causal} U={U}", flush=True)
        o, lse = up.attn_fwd(q, k, v, causal=causal, U=U)
        got = (o, lse) + tuple(up.attn_bwd(q, k, v, o, lse, do, causal=causal, U=U))
        torch.cuda.synchronize()
        if first is None:
            first = got
        for a, b in zip(first, got):
            assert torch.equal(_bits(a), _bits(b)), U
    b = B - 1
    _check(q[b], k[b], v[b], do[b], *(t[b] for t in first), causal, S)


def test_long_backward_of_many_heads():
    """36 heads: at U = 1 the row terms of all of them do not fit and dQ runs chunk by
    chunk; at U = 2 they do.  Bitwise equal, and a head of each group against the
    oracle (a group's dk, dv sum all 18 heads)."""
    up = _upipe()
    S, Hq, Hkv = 65600, 36, 2
    q, k, v, do = (t[0] for t in _qkvd(1, S, Hq, Hkv, 36))
    outs = []
    for U in (1, 2):
        print(f"many heads S={S} Hq={Hq} U={U}", flush=True)
        o, lse = up.attn_fwd(q, k, v, U=U)
        outs.append((o, lse) + tuple(up.attn_bwd(q, k, v, o, lse, do, U=U)))
        torch.cuda.synchronize()
    for a, b in zip(*outs):
        assert torch.equal(_bits(a), _bits(b))
    o, lse, dq, dk, dv = outs[0]
    for g in range(Hkv):
        h = slice(18 * g, 18 * g + 18)
        _check(q[:, h], k[:, g:g + 1], v[:, g:g + 1], do[:, h], o[:, h], lse[h], dq[:, h],
               dk[:, g:g + 1], dv[:, g:g + 1], True, g)


def test_backward_packs_keys_beyond_32_bit_offsets():
    """2^18 rows of 64 key/value heads: one head's rows span 2^32 bytes, so keys and
    values are packed; each head is bitwise what it is alone, where its rows are
    read in place."""
    up = _upipe()
    S, H = 1 << 18, 64
    q, k, v, do = (t[0] for t in _qkvd(1, S, H, H, 64))
    print(f"packed keys S={S} H={H} forward", flush=True)
    o, lse = up.attn_fwd(q, k, v, U=1)
    print("  backward", flush=True)
    got = up.attn_bwd(q, k, v, o, lse, do, U=1)
    torch.cuda.synchronize()
    for h in (0, 31, 63):
        x = [t[:, h:h + 1].contiguous() for t in (q, k, v, o, do)]
        o1, l1 = up.attn_fwd(*x[:3], U=1)
        assert torch.equal(_bits(o1), _bits(x[3])) and torch.equal(_bits(l1[0]), _bits(lse[h])), h
        one = up.attn_bwd(*x[:3], x[3], lse[h:h + 1].contiguous(), x[4], U=1)
        torch.cuda.synchronize()
        for a, b in zip(got, one):
            assert torch.equal(_bits(a[:, h]), _bits(b[:, 0])), h
