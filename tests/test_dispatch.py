"""The rule that sends a multi-frame call to the two passes or to the segment decoders (csrc/pb_lines.hpp, host code without
HIP), compiled by itself: the sizes that the GPU tests name as lying on one side do, every row shape of the segment decoders
has a call that reaches it, longer lists never widen the rule, and what was measured as slower in two passes stays out."""
import ctypes
import os
import shutil
import subprocess

import pytest

from sizes import LINES, SEGMENTS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FEW = 3000  # states of the trees that the GPU tests build


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("lines")
    (d / "lines.cpp").write_text('#include "pb_lines.hpp"\nextern "C" int two(int V, int T, int B, int mode, int n) '
                                 '{ return pb::rows_pay(V, T, B, mode, n) ? 1 : 0; }\n')
    so = str(d / "lines.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2508_07014_amd", "csrc"), str(d / "lines.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so).two


@pytest.mark.parametrize("V,T,B,two", LINES)
def test_lines(rule, V, T, B, two):
    assert tuple(m for m in (0, 1, 2) if rule(V, T, B, m, FEW)) == two


@pytest.mark.parametrize("V", sorted(SEGMENTS))
def test_segment_calls(rule, V):
    T, B = SEGMENTS[V]
    assert not any(rule(V, T, B, m, FEW) for m in (0, 1, 2))


def test_longer_lists_never_widen_the_rule(rule):
    for V in (128, 256, 257, 384, 512, 768, 1000, 1024, 1025, 1152, 1280, 2000, 4095, 4096, 8192, 16384, 20000):
        for T in (1, 40, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049):
            for B in (1, 2, 4, 8, 16, 17, 64, 128, 512, 2000):
                for mode in (0, 1, 2):
                    few, some, many = (rule(V, T, B, mode, n) for n in (16384, 49152, 1 << 20))
                    assert few >= some >= many, (V, T, B, mode)
                    assert mode == 2 or rule(V, T, B, 2, 1000) >= rule(V, T, B, mode, 1000), (V, T, B, mode)


# Slower in two passes over random rows, bf16 logits and phrases (geometric mean 1.1 .. 2.1): more than 1024 frames
@pytest.mark.parametrize("V,T,B,mode,states", [(1152, 2000, 1, 0, 9500), (1152, 2000, 1, 1, 80000), (1280, 2000, 2, 0, 27000),
                                               (2000, 2000, 1, 0, 80000), (2000, 2000, 3, 1, 27000), (1025, 2000, 8, 2, 80000),
                                               (1280, 2000, 50, 2, 27000), (2000, 2000, 8, 2, 27000)])
def test_slower_calls_stay_out(rule, V, T, B, mode, states):
    assert not rule(V, T, B, mode, states)


# Faster in two passes than in segments, long lists or not (0.5 .. 0.75 of the time): calls a tighter rule lost
@pytest.mark.parametrize("V,T,B,mode,states", [(5569, 755, 23, 1, 47368), (385, 163, 9, 1, 16736), (3521, 731, 2, 1, 22695), (9537, 522, 20, 0, 21557),
                                               (960, 155, 5, 1, 24650), (705, 228, 5, 1, 43014), (577, 130, 14, 1, 39255), (7525, 896, 14, 2, 16747)])
def test_faster_calls_stay_in(rule, V, T, B, mode, states):
    assert rule(V, T, B, mode, states)
