"""Which items a workgroup walks (csrc/xcd_range.h), compiled for the host."""
import ctypes
import os
import shutil
import subprocess

import pytest

_CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2003_08646_amd", "csrc")
_CXX = shutil.which("g++") or shutil.which("c++")

_SRC = """
#define __device__
#define __forceinline__ inline
namespace lance { namespace dev {
inline int fast_div(int x, unsigned magic) { return magic == 0 ? x : (int)((unsigned long long)(unsigned)x * magic >> 32); }
}}
#include "xcd_range.h"
extern "C" void items(int n, int block, int blocks, int* out) {
  const unsigned magic = blocks <= 1 ? 0u : (unsigned)(((1ULL << 32) + blocks - 1) / blocks);
  const lance::dev::XcdRange r(n / blocks, n % blocks, magic, block, blocks);
  out[0] = r.first; out[1] = r.end; out[2] = r.step;
}
"""


@pytest.fixture(scope="module")
def items(tmp_path_factory):
    if _CXX is None:
        pytest.skip("needs a host compiler")
    d = tmp_path_factory.mktemp("xcd")
    shutil.copy(os.path.join(_CSRC, "xcd_range.h"), d)
    (d / "lance_device.h").write_text("#pragma once\n")               # what it needs is in _SRC
    (d / "xcd.cpp").write_text(_SRC)
    subprocess.run([_CXX, "-std=c++17", "-shared", "-fPIC", str(d / "xcd.cpp"), "-o", str(d / "xcd.so")], check=True)
    f = ctypes.CDLL(str(d / "xcd.so")).items

    def walk(n, block, blocks):
        out = (ctypes.c_int * 3)()
        f(n, block, blocks, out)
        return range(out[0], out[1], out[2])
    return walk


@pytest.mark.parametrize("blocks", [1, 2, 7, 8, 9, 15, 16, 100, 255, 256, 511, 512, 1023, 1024])
def test_every_item_once_and_every_round_on_all_dies(items, blocks):
    for n in (blocks, blocks + 1, blocks + 7, blocks + blocks // 3, 2 * blocks - 1, 2 * blocks, 5 * blocks + 3):
        own = [items(n, b, blocks) for b in range(blocks)]
        assert sorted(i for w in own for i in w) == list(range(n))
        assert all(w[0] == w.start for w in own)                       # at least one to a workgroup
        assert max(len(w) for w in own) <= -(-n // blocks) + 1         # (a die with a remainder: one round more)
        assert n % blocks or max(len(w) for w in own) == n // blocks
        for x in range(min(blocks, 8)):
            die = [w for b, w in enumerate(own) if b % 8 == x]
            done = sorted(i for w in die for i in w)
            assert done == list(range(done[0], done[-1] + 1))          # one contiguous range
            assert abs(len(done) - n * len(die) / blocks) < 1 + 1e-9   # as long as its workgroups


def test_large_counts_do_not_overflow(items):
    n = 1 << 29
    assert items(n, 511, 512)[-1] == n - 1 and items(n, 0, 512)[0] == 0
