"""How many waves of the small-channel kernel share 64 tiles (csrc/share_rule.h), compiled for the host."""
import ctypes
import os
import shutil
import subprocess

import pytest

from test_gpu_plans import _C16_SHARED

_CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2003_08646_amd", "csrc")
_CXX = shutil.which("g++") or shutil.which("c++")

_SRC = """
#include "share_rule.h"
extern "C" int split(long long tiles, int C, int K, int nhwc, long long y_bytes) {
  return lance::c16_split(tiles, C, K, nhwc, y_bytes);
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    if _CXX is None:
        pytest.skip("needs a host compiler")
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(_SRC)
    subprocess.run([_CXX, "-std=c++17", "-shared", "-fPIC", "-I", _CSRC, str(d / "rule.cpp"), "-o", str(d / "rule.so")], check=True)
    f = ctypes.CDLL(str(d / "rule.so")).split
    f.argtypes, f.restype = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_longlong], ctypes.c_int

    def of(N, C, K, H, W, pad, nhwc):
        Ho, Wo = H + 2 * pad - 2, W + 2 * pad - 2
        return f(N * -(-Ho // 2) * -(-Wo // 2), C, K, nhwc, 4 * N * K * Ho * Wo)
    return of


@pytest.mark.parametrize("shape", _C16_SHARED, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_b%d%s_%d" % (s[:7] + ("_nhwc" if s[7] else "",) + s[8:]))
def test_the_gpu_tests_shapes_are_divided_as_they_claim(split, shape):
    N, C, K, H, W, pad, bits, nhwc, waves = shape
    assert split(N, C, K, H, W, pad, nhwc) == waves


@pytest.mark.parametrize("shape,waves", [
    ((16, 3, 64, 224, 224, 1, False), 1), ((16, 3, 64, 224, 224, 1, True), 1),      # every compute unit has work
    ((959, 3, 294, 16, 16, 1, False), 1), ((803, 16, 209, 20, 20, 1, False), 1),    # and Y exceeds the last-level cache
    ((229, 15, 872, 24, 24, 1, True), 1), ((472, 2, 763, 19, 19, 1, False), 4),
])
def test_not_where_the_chip_is_full(split, shape, waves):
    assert split(*shape) == waves
