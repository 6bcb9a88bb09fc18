"""Slices of a batched preconditioner application: every packed offset and every
grid index of a slice stays in range, and no slice is smaller than it has to be."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_21410_amd", "csrc")


@pytest.fixture(scope="module")
def batch_slice(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("slice")
    src, so = d / "s.cpp", d / "s.so"
    src.write_text('#include "cheb_host.h"\nextern "C" int f(int a, int b, int c) '
                   "{ const int m[3] = {a, b, c}; return cheb::batch_slice(m); }\n")
    subprocess.run([cxx, "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    return ctypes.CDLL(str(so)).f


@pytest.mark.parametrize("m", [(1, 1, 1), (15, 15, 15), (31, 33, 35), (127, 127, 127), (128, 128, 128), (128, 1, 3),
                               (511, 511, 511)])
def test_batch_slice(m, batch_slice):
    k, each = batch_slice(*m), m[0] * m[1] * m[2]
    assert 1 <= k <= 65535
    assert k * each < 2 ** 31
    assert k == 65535 or (k + 1) * each >= 2 ** 31
