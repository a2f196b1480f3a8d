"""Which kernels count and list the tetrahedra: the rule alone, compiled for
the host.  The measured points of its table, and results that hold no
triangles (builds up to the edges), whose links may be of any size."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1809_04424_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src, lib = str(d / "rule.cpp"), str(d / "rule.so")
    with open(src, "w") as f:
        f.write('#include "vr_tetra.h"\n'
                'extern "C" int by_wave(int w, long long n, long long K, long long T) '
                '{ return tet_by_wave(w != 0, n, K, T); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    f = ctypes.CDLL(lib).by_wave
    f.argtypes = [ctypes.c_int] + [ctypes.c_longlong] * 3
    return lambda write, n, K, T: bool(f(write, n, K, T))


@pytest.mark.parametrize("n,K,per,count,write", [
    (400, 11975, 12, True, True), (1000, 24975, 9, True, True), (300, 11212, 18, False, True),
    (150, 11175, 49, False, False), (1000, 99900, 50, False, True), (1024, 157132, 57, False, True),
    (400, 79800, 133, False, False), (1025, 24975, 9, False, False), (400, 4095, 9, False, False)])
def test_measured_points(rule, n, K, per, count, write):
    assert rule(0, n, K, per * K) == count
    assert rule(1, n, K, per * K) == write


@pytest.mark.parametrize("n,K", [(400, 79800), (1000, 99900), (150, 11175)])
def test_triangles_not_counted(rule, n, K):
    assert not rule(0, n, K, 0) and not rule(1, n, K, 0)
