"""The patch loader of the few-tile and weight-only kernels (csrc/tile_loader.h) on the CPU: the header
is compiled for the host against buffer loads that check every address.  Over small images, paddings,
batches and channel counts no load of an existing row may have a negative (wrapped) offset, start in
front of the tensor, or cross its end where the lane's value counts; masked patches hold the padded
image."""
import os
import re
import shutil
import subprocess

import pytest

_CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2003_08646_amd", "csrc")
_CLANG = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")) if c and os.path.exists(c)), None)

_STUB = r"""
#pragma once
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <vector>
#define __device__
#define __forceinline__ inline
using std::min; using std::max;
inline unsigned long long __ballot(bool b) { return b; }
inline unsigned __float_as_uint(float f) { unsigned u; memcpy(&u, &f, 4); return u; }
inline float __uint_as_float(unsigned u) { float f; memcpy(&f, &u, 4); return f; }
inline float __int_as_float(int u) { return __uint_as_float((unsigned)u); }
typedef int i4 __attribute__((ext_vector_type(4)));
typedef int i2 __attribute__((ext_vector_type(2)));
struct Rsrc { const char* base; unsigned extent; };
#define __amdgpu_buffer_rsrc_t Rsrc
extern const char *x_first, *x_end;
extern bool counts;  // the lane's channel exists
extern const char* bad;
inline Rsrc __builtin_amdgcn_make_buffer_rsrc(char* b, int, unsigned extent, int) { return {b, extent}; }
// dwords off .. off+n-1 as the hardware sees them: beyond the extent they read 0
template <int N> inline void fetch(Rsrc r, unsigned off, int* v) {
  if (r.base + r.extent != x_end) bad = "extent";
  if (off < r.extent && off + 4ull * N > r.extent && counts) bad = "a load that counts crosses the tensor's end";
  for (int i = 0; i < N; i++) {
    v[i] = 0;
    if (off + 4ull * i + 4 > r.extent) continue;
    const char* at = r.base + off + 4 * i;
    if (at < x_first) bad = "in front of the tensor";
    else memcpy(&v[i], at, 4);
  }
}
inline i4 __builtin_amdgcn_raw_buffer_load_b128(Rsrc r, unsigned o, int, int) { int v[4]; fetch<4>(r, o, v); return i4{v[0], v[1], v[2], v[3]}; }
inline i2 __builtin_amdgcn_raw_buffer_load_b64(Rsrc r, unsigned o, int, int) { int v[2]; fetch<2>(r, o, v); return i2{v[0], v[1]}; }
inline int __builtin_amdgcn_raw_buffer_load_b32(Rsrc r, unsigned o, int, int) { int v[1]; fetch<1>(r, o, v); return v[0]; }
"""

_MAIN = r"""
#include "tile_loader.h"
const char *x_first, *x_end, *bad = nullptr;
bool counts;
using namespace lance::pos;

template <int M, int LOAD> long check(int N, int C, int H, int W, int pad) {
  constexpr int A = M + 2;
  constexpr bool nhwc = LOAD == kNhwc1;
  const int Ho = H + 2 * pad - 2, Wo = W + 2 * pad - 2;
  if (Ho <= 0 || Wo <= 0 || (LOAD == kRowsEdge && (pad != 1 || W % M))) return 0;
  const int th = (Ho + M - 1) / M, tw = (Wo + M - 1) / M, P = N * th * tw;
  std::vector<float> buf(64 + (size_t)N * C * H * W + 64, -7.0f);
  float* x = buf.data() + 64;
  const size_t count = (size_t)N * C * H * W;
  for (size_t i = 0; i < count; i++) x[i] = (float)(i + 1);
  x_first = (const char*)x; x_end = (const char*)(x + count);
  const TileGeo g{x, (unsigned)(count * 4), N, C, H, W, pad, P, th, tw};
  long loads = 0;
  for (int p = 0; p < P; p++)
    for (int dl = 0; dl < (nhwc ? 16 : 4); dl++) {
      TileLoader<M, LOAD> tl;
      tl.setup(g, p, dl);
      const int ty = p / tw % th, tx = p % tw, n = p / tw / th;
      for (int any = 0; any < 2; any++) {  // another lane of the wave may set the limits, too
        if (any) { tl.first_end = std::max(tl.first_end, 1); tl.last_begin = C - 4; }
        for (int cu0 = 0; cu0 < C + 4; cu0 += nhwc ? 16 : 4) {
          const int cu = std::min(cu0, C - 1);  // as the kernels clamp it
          counts = cu0 + dl < C;
          float b[A * A], d[A][A];
          tl.load(g, cu, b);
          tl.mask(b, d);
          loads++;
          for (int r = 0; r < A; r++) {
            if (!nhwc && tl.rowoff[r] > kOutside) bad = "negative offset";
            for (int s = 0; s < A; s++) {
              const int iy = ty * M - pad + r, ix = tx * M - pad + s, c = cu0 + dl;
              const bool in = iy >= 0 && iy < H && ix >= 0 && ix < W;
              const float want = !in ? 0.0f : x[nhwc ? (((size_t)n * H + iy) * W + ix) * C + std::min(c, C - 1)
                                                     : (((size_t)n * C + std::min(c, C - 1)) * H + iy) * W + ix];
              if (counts && d[r][s] != want) bad = "value";
            }
          }
          if (bad) {
            printf("m%d load%d N%d C%d %dx%d pad%d tile %d dl %d cu %d: %s\n", M, LOAD, N, C, H, W, pad, p, dl, cu, bad);
            exit(1);
          }
        }
      }
    }
  return loads;
}

int main() {
  long loads = 0;
  const int sizes[][2] = {{1, 1}, {1, 2}, {1, 3}, {3, 1}, {2, 2}, {1, 7}, {2, 3}, {2, 4}, {4, 2}, {8, 1}, {1, 9}, {3, 4}, {4, 4}, {5, 3}, {6, 8}};
  for (auto& s : sizes)
    for (int pad : {0, 1, 2, 3, 4, 5, 6, 9, 13, 14, 20})
      for (int N : {1, 2, 3})
        for (int C : {1, 2, 3, 4, 5, 8, 9, 21}) {
          loads += check<2, kRowsEdge>(N, C, s[0], s[1], pad) + check<2, kRowsAny>(N, C, s[0], s[1], pad) + check<2, kNhwc1>(N, C, s[0], s[1], pad);
          loads += check<4, kRowsEdge>(N, C, s[0], s[1], pad) + check<4, kRowsAny>(N, C, s[0], s[1], pad) + check<4, kNhwc1>(N, C, s[0], s[1], pad);
        }
  printf("%ld loads\n", loads);
}
"""


@pytest.mark.skipif(_CLANG is None, reason="needs clang's vector types")
def test_every_address_lies_in_the_tensor(tmp_path):
    with open(os.path.join(_CSRC, "tile_loader.h")) as f:
        # (the register constraints of the GPU's assembly)
        (tmp_path / "tile_loader.h").write_text(re.sub(r"asm volatile\([^;]*\);", "", f.read()))
    (tmp_path / "lance_device.h").write_text(_STUB)
    (tmp_path / "main.cpp").write_text(_MAIN)
    exe = str(tmp_path / "loader")
    subprocess.run([_CLANG, "-std=c++17", "-O2", "-fno-strict-aliasing", "-w", str(tmp_path / "main.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
