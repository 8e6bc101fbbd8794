"""Scratch memory of the built kernels: those of the small coordination classes whose
registers suffice have none, so nothing that they keep per item and per lane is a
struct in memory (written in branches it was: 20 bytes a lane in each of them, every
use of a field a load).
"""
import os
import re

import pytest

from paper_1909_11474_amd import build as B


def scratch_bytes():
    """Kernel name -> private segment bytes a lane, from the code objects' metadata
    (MessagePack, keys in order: .name comes before .private_segment_fixed_size)."""
    blob = open(B.LIB, "rb").read()
    out = {}
    for m in re.finditer(rb"\.name(?:[\xa0-\xbf]|\xd9.|\xda..)(_ZN2mt\w+).{0,4}?\.private_segment_fixed_size(...)",
                         blob, re.S):
        v = m[2]
        out[m[1].decode()] = v[0] if v[0] < 0x80 else v[1] if v[0] == 0xcc else v[1] << 8 | v[2]
    return out


def test_small_classes_have_no_scratch():
    if not os.path.exists(B.LIB):
        pytest.skip("library not built")
    s = {re.match(r"_ZN2mt9(k_\w+?)I(.*?)EEEv", n)[0]: v for n, v in scratch_bytes().items()
         if re.match(r"_ZN2mt9(k_batched|k_adjoint)I", n)}
    assert len(s) >= 30 and max(s.values()) > 100          # the larger classes do spill
    # k_batched<S, mode, class, ...>: float fitness of class 6, evaluation of class 4;
    # k_adjoint<S, class, ...>: float class 4 of the Tersoff form (the minimal form's is held
    # to 128 registers for four wavefronts a SIMD, and spills for that)
    small = [n for n in s if re.search(r"k_batchedI(fLi0ELi6|fLi1ELi4)E|k_adjointIfLi4ELb1E", n)]
    assert len(small) == 5
    assert {n: s[n] for n in small if s[n]} == {}


def test_float_evaluation_takes_no_moments():
    """The float evaluation kernel of up to 16 neighbours holds no angular moments, whose
    registers would go to scratch (1,080 bytes a lane or more with them, 832 without)."""
    if not os.path.exists(B.LIB):
        pytest.skip("library not built")
    s = scratch_bytes()
    n, = [n for n in s if n.startswith("_ZN2mt9k_batchedIfLi1ELi16ELb0E")]
    assert 0 < s[n] < 1000
