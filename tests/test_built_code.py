"""What the built GPU code may not contain, read from the library's own disassembly."""
import glob
import os
import re
import shutil
import subprocess

import pytest

_LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2003_08646_amd", "liblance.so")
_OBJDUMP = next((c for c in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if c and os.path.exists(c)), None)


@pytest.fixture(scope="module")
def buffer_stores(tmp_path_factory):
    """(kernel, line) of every buffer store of the library."""
    if _OBJDUMP is None:
        pytest.skip("needs llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    shutil.copy(_LIB, d / "lib.so")
    subprocess.run([_OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    images = glob.glob(str(d / "*gfx950"))
    assert images
    stores = []
    for image in images:
        asm = subprocess.run([_OBJDUMP, "-d", "--no-show-raw-insn", image], check=True, capture_output=True, text=True).stdout
        kernel = ""
        for line in asm.splitlines():
            if line.endswith(">:"):
                kernel = line.split("<")[1][:-2]
            elif "buffer_store_" in line:
                stores.append((kernel, line))
    assert stores
    return stores


def test_wide_buffer_stores_have_no_register_as_scalar_offset(buffer_stores):
    """A buffer store of more than 8 bytes must not be followed at once by a write of its data registers.  The
    compiler keeps that rule only where the scalar offset is a constant, but on gfx950 it holds with a register
    there too (the first words of stored rows came from the next row)."""
    wide = [(k, re.search(r"dwordx[34] v\[[^]]*\], (?:v\d+|off), s\[[^]]*\], (\S+)", l)) for k, l in buffer_stores]
    wide = [(k, m.group(1)) for k, m in wide if m]
    assert wide
    assert not [w for w in wide if re.match(r"s\d|m0|ttmp|vcc", w[1])]


@pytest.mark.parametrize("name", ["conv_fused_c16_kernel", "conv_fused_c16_shared_kernel", "conv_fused_pairs_nhwc_c64_kernel",
                                  "conv_fused_pairs_nhwc_c128_kernel", "conv_fused_any_pairs_nhwc_c64_kernel",
                                  "conv_fused_any_pairs_nhwc_c128_kernel"])
def test_kernels_of_cached_stores(buffer_stores, name):
    """Cached and non-temporal stores in one kernel cost the layers whose stores are cached: each of these kernels
    has a form without non-temporal stores (last template argument)."""
    forms = {}
    for kernel, line in buffer_stores:
        if name in kernel:
            m = re.search(r"I((?:L\w\d+E)*?)(Lb[01]E)?E", kernel[kernel.index(name):])
            forms.setdefault(m.group(1), {}).setdefault(m.group(2), set()).add(" nt" in line)
    assert forms and any("Lb1E" in f for f in forms.values())
    for f in forms.values():
        assert f["Lb0E"] == {False}
        assert True in f.get("Lb1E", {True})
