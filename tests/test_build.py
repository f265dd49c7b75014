"""What the kernels' sources rely on in the code that the compiler makes of them."""

import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2602_21196_amd import build as B

COPYING = ("attn_bwd.hip", "attn_fwd.hip", "gemm.hip")   # use copy_b128 and its like


def _assembly(name):
    cmd = [B.HIPCC, *B.COMMON, "-x", "hip", "-S", "--cuda-device-only",
           os.path.join(B.CSRC, name), "-o", "-"]
    return subprocess.run(cmd, capture_output=True, text=True, check=True).stdout


def _outside_asm(text):
    """Instructions that the compiler made itself (inline assembly stands between
    ;;#ASMSTART and ;;#ASMEND), without comments."""
    text = re.sub(r";;#ASMSTART.*?;;#ASMEND", "", text, flags=re.S)
    return [line.split(";")[0] for line in text.splitlines()
            if line.strip() and line.startswith("\t") and not line.startswith("\t.")]


def test_inline_assembly_is_told_apart():
    text = "\ts_nop 0\n\t;;#ASMSTART\n\ts_mov_b32 m0, s1\n\t;;#ASMEND\n\ts_mov_b32 m0, s2 ; x\n"
    assert [line.strip() for line in _outside_asm(text)] == ["s_nop 0", "s_mov_b32 m0, s2"]


def test_only_the_written_out_copies_touch_m0():
    """The inline copies write m0, which the compiler does not let a clobber list
    name: none of the instructions around them may use it."""
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    with ThreadPoolExecutor(len(COPYING)) as pool:
        texts = list(pool.map(_assembly, COPYING))
    for name, text in zip(COPYING, texts):
        assert re.search(r"s_mov_b32 m0,", text), name
        found = [line.strip() for line in _outside_asm(text) if re.search(r"\bm0\b", line)]
        assert not found, (name, found[:5])
