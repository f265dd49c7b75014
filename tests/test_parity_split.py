"""GPU parity where the launch rule changes: the attention forward splits the
keys of a stage into 1, 2 or 4 parts by the number of 256-row query blocks
times heads, and packs keys and values only when one head's token-major rows
span 2^32 bytes.  Query counts end one row into a block, on it and before it;
the key ranges are short, so the oracle stays cheap."""

import numpy as np
import pytest
import torch

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
