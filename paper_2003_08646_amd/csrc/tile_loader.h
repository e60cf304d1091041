// The (m+2)x(m+2) patch of one tile and one channel per lane, for kernels whose lanes take 16 tiles
// x 4 channels (NCHW) or 4 tiles x 16 channels (NHWC).  X is below 2^31 bytes.
//
// NCHW patches are loaded by rows (one 16-byte load, for m = 4 also an 8-byte one, at any 4-byte
// alignment) whatever the padding and the width: pixels of a neighbouring row are masked away
// afterwards, rows without a pixel of the image have an offset beyond the buffer.  A row that has one
// starts at most m+1 pixels before its plane and ends at most m+1 after it: with the guard in front of
// the buffer's base no offset is negative, and in images of kTinyImage pixels or more the row stays
// within the neighbouring planes.  Only where such a load would start before the tensor or end after it
// (its first and last plane; any plane of a smaller image) the wave takes pixel loads.
#pragma once
#include "lance_device.h"

namespace lance {
namespace pos {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

// How the patches are loaded.
constexpr int kRowsEdge = 0;  // NCHW by rows; only the edge columns can be outside the image
constexpr int kRowsAny = 1;   // NCHW by rows; any column can be outside
constexpr int kNhwc1 = 2;     // NHWC, 4-byte loads
constexpr int kNhwc4 = 3;     // NHWC, 16-byte loads of four channels (C a multiple of 4)

constexpr unsigned kOutside = 0x80000000u;
constexpr unsigned kGuard = 20;   // bytes: five pixels, the most a row of F(4x4) starts before its plane
constexpr int kTinyImage = 8;     // pixels: more than those five

__device__ __forceinline__ v4f load_b128(const char* base, unsigned extent, unsigned off) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, extent, 0x00020000);
  return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ v2f load_b64(const char* base, unsigned extent, unsigned off) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, extent, 0x00020000);
  return __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ float load_b32(const char* base, unsigned extent, unsigned off) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, extent, 0x00020000);
  return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
struct TileGeo {
  const float* x;
  unsigned x_bytes;
  int N, C, H, W, pad, P, th, tw;
};

template <int M, int LOAD>
struct TileLoader {
  static constexpr int A = M + 2;
  static constexpr bool kNhwc = LOAD == kNhwc1 || LOAD == kNhwc4;
  unsigned rowoff[A];  // byte offset of the patch row's first pixel (channel 0, NCHW: channel dl)
  unsigned cmask[A];   // all ones where the patch column lies inside the image
  int ix0, dl, C, W;
  // Channels below first_end, and from last_begin on: a row load of some lane may leave the tensor (in
  // its first or last plane; in images of fewer than kTinyImage pixels in any).
  int first_end, last_begin;

  // p: the lane's tile (clamped); dl: its channel relative to the wave's (NCHW: below 4)
  __device__ __forceinline__ void setup(const TileGeo& g, int p, int dl_) {
    const int tx = p % g.tw, t2 = p / g.tw;
    const int ty = t2 % g.th, n = t2 / g.th;
    const int iy0 = ty * M - g.pad;
    const unsigned HW = (unsigned)g.H * (unsigned)g.W;
    ix0 = tx * M - g.pad;
    dl = dl_; C = g.C; W = g.W;
    bool first = false, last = false;
    const bool cols = LOAD != kRowsAny || (ix0 > -A && ix0 < W);  // a row load meets the image
#pragma unroll
    for (int r = 0; r < A; r++) {
      const int iy = iy0 + r;
      const bool ok = cols && iy >= 0 && iy < g.H;
      if constexpr (kNhwc) {
        rowoff[r] = ok ? (((unsigned)n * (unsigned)g.H + (unsigned)iy) * (unsigned)W + (unsigned)ix0) *
                             (unsigned)C * 4u
                       : kOutside;
      } else {
        rowoff[r] = ok ? (((unsigned)n * (unsigned)C + (unsigned)dl) * HW + (unsigned)iy * (unsigned)W +
                          (unsigned)ix0) * 4u + kGuard
                       : kOutside;
        first |= ok && n == 0 && iy * W + ix0 < 0;
        last |= ok && n == g.N - 1 && iy * W + ix0 + A > (int)HW;
      }
    }
#pragma unroll
    for (int s = 0; s < A; s++) cmask[s] = (ix0 + s >= 0 && ix0 + s < W) ? 0xFFFFFFFFu : 0u;
    first_end = HW < (unsigned)kTinyImage ? C : (__ballot(first) != 0 ? 1 : 0);
    last_begin = __ballot(last) != 0 ? C - 4 : C;
  }

  // Channel cu + dl of the lane's patch (cu wave-uniform, below C).  NCHW lanes whose channel does not
  // exist get anything finite-or-not that lies inside the tensor, or zero; NHWC ones channel C-1.
  __device__ __forceinline__ void load(const TileGeo& g, int cu, float (&b)[A * A]) const {
    const char* base = reinterpret_cast<const char*>(g.x);
    if constexpr (LOAD == kNhwc1) {
      const unsigned c4 = (unsigned)min(cu + dl, C - 1) * 4u, px = (unsigned)C * 4u;
#pragma unroll
      for (int r = 0; r < A; r++)
#pragma unroll
        for (int s = 0; s < A; s++) b[r * A + s] = load_b32(base, g.x_bytes, rowoff[r] + (c4 + (unsigned)s * px));
    } else if constexpr (LOAD != kNhwc4) {
      const unsigned plane = (unsigned)cu * (unsigned)g.H * (unsigned)g.W * 4u;
      base += (size_t)plane;
      base -= kGuard;
      const unsigned extent = g.x_bytes + kGuard - plane;
      if (cu < first_end || cu >= last_begin) {
        // (offsets from a copy the compiler cannot see through: formed here, not kept in registers)
        int ix = ix0;
        asm volatile("" : "+v"(ix));
#pragma unroll
        for (int r = 0; r < A; r++)
#pragma unroll
          for (int s = 0; s < A; s++)
            b[r * A + s] = load_b32(base, extent, (ix + s >= 0 && ix + s < W) ? rowoff[r] + 4u * s : kOutside);
      } else {
#pragma unroll
        for (int r = 0; r < A; r++) {
          const v4f v = load_b128(base, extent, rowoff[r]);
          b[r * A] = v[0]; b[r * A + 1] = v[1]; b[r * A + 2] = v[2]; b[r * A + 3] = v[3];
          if constexpr (A == 6) {
            const v2f w = load_b64(base, extent, rowoff[r] + 16u);
            b[r * A + 4] = w[0]; b[r * A + 5] = w[1];
          }
        }
      }
    }
  }
  // Channels c .. c+3 of every pixel (kNhwc4; c + 3 < C).
  __device__ __forceinline__ void load4(const TileGeo& g, int c, v4f (&w)[A * A]) const {
    const unsigned c4 = (unsigned)c * 4u, px = (unsigned)C * 4u;
#pragma unroll
    for (int r = 0; r < A; r++)
#pragma unroll
      for (int s = 0; s < A; s++)
        w[r * A + s] = load_b128(reinterpret_cast<const char*>(g.x), g.x_bytes,
                                 rowoff[r] + (c4 + (unsigned)s * px));
  }
  // d = the patch with the pixels outside the image zeroed
  __device__ __forceinline__ void mask(const float (&b)[A * A], float (&d)[A][A]) const {
#pragma unroll
    for (int r = 0; r < A; r++)
#pragma unroll
      for (int s = 0; s < A; s++)
        d[r][s] = (LOAD == kRowsEdge && s > 0 && s < A - 1)
                      ? b[r * A + s]
                      : __uint_as_float(__float_as_uint(b[r * A + s]) & cmask[s]);
  }
};

}  // namespace pos
}  // namespace lance
