// Transform + quantize of F(2x2,3x3) tiles into LDS, two horizontally adjacent tiles per lane:
// v^ = Q(B^T d B) (Algorithm 1; Eq. 7) formed in registers, the signed 8-bit codes written as code
// rows [E][TILES][64 B].  NCHW tensors, pad 1, image widths that are multiples of 4: a lane's pair of tiles 2q, 2q+1 of a tile row then
// owns the aligned 16-byte segment 4q .. 4q+3 of each of its four image rows.
//
// What it saves against one tile per lane (quant_phase.h): one 16-byte load per row for two tiles
// instead of two unaligned ones (the vector memory unit takes a wave-wide load every 16 to 25
// cycles, and the transform phase was as much bound by that as by its arithmetic), a column pass
// over four pixel columns instead of eight, no zeroing of edge pixels before the transform, and
// no special case at the ends of the tensor: every load lies inside an image row or is out of the
// buffer's range as a whole.  The column left of the segment is the left neighbour's last one,
// already through the column pass there (the same operations on the same values), and comes by a
// DPP move inside the group of 16 lanes; the two lanes at the ends of a group load the one column
// that they cannot get that way themselves (a 4-byte load per row, out of range for the others).
//
// Called by all 512 threads (8 waves) of a workgroup.  A lane owns the pair lane % PAIRS and one
// dword of its wave's 16-byte chunk of the code rows: channels c_base + 4*chunk + d + 16b, b = 0..3
// the byte, d = dbase + lane / PAIRS the dword.  LDS row of tile s (0 left, 1 right) of pair i:
// PAIRS * s + i; the 16-byte chunk c of row r is stored at chunk c ^ row_swizzle_mfma32(r).
#pragma once
#include "lance_device.h"

namespace lance {
namespace dev {

// What the kernel knows about the tensor; divisors as in fast_div.
struct PairGeo {
  const float* x;
  int C, H, W, th, npr, pairs, bits;  // npr: pairs per tile row; pairs: of the whole batch
  unsigned th_magic, npr_magic;
  unsigned reach;  // extent of the buffer descriptors: bytes from a plane of a block's first image
};

// B8: 8-bit codes.  FULL: all 64 channels of every block exist.
template <bool B8, bool FULL, int PAIRS>
struct PairPhase {
  typedef float f4 __attribute__((ext_vector_type(4)));
  static constexpr int E = 16, kSteps = 4, kTiles = 2 * PAIRS;
  static constexpr unsigned kOutside = 0x80000000u;  // extents are below 2^31

  struct Pixels {
    f4 own[4];   // the segment's four pixels of each row
    float edge;  // lanes 0..3 of a group: rows 0..3 of the column left of the group; 4..7: right of it
  };
  unsigned own_off[4], edge_off;
  bool left_edge, right_edge;
  const char* base;    // first image of the block
  int c_wave, group;   // the wave's first channel (+ 16 for each step); lane / PAIRS

  __device__ __forceinline__ static void locate(const PairGeo& g, int p, int* q, int* ty, int* n) {
    const int t2 = fast_div(p, g.npr_magic);
    *q = p - t2 * g.npr;
    *n = fast_div(t2, g.th_magic);
    *ty = t2 - *n * g.th;
  }
  // block: PAIRS consecutive pairs of the batch
  __device__ __forceinline__ void setup(const PairGeo& g, int block, int c_first, int lane) {
    const int p0 = block * PAIRS;
    c_wave = c_first;
    group = lane / PAIRS;
    const unsigned HW = (unsigned)g.H * (unsigned)g.W;
    const int n0 = fast_div(fast_div(p0, g.npr_magic), g.th_magic);
    base = reinterpret_cast<const char*>(g.x + (size_t)n0 * g.C * HW);
    int q, ty, n;
    locate(g, min(p0 + lane % PAIRS, g.pairs - 1), &q, &ty, &n);
    left_edge = q == 0;
    right_edge = q == g.npr - 1;
    const unsigned plane0 = FULL ? (unsigned)group * HW : 0u;
    unsigned img = (unsigned)(n - n0) * (unsigned)g.C * HW + plane0;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int y = 2 * ty - 1 + r;
      own_off[r] = y >= 0 && y < g.H ? (img + (unsigned)y * (unsigned)g.W + 4u * (unsigned)q) * 4u : kOutside;
    }
    const int i = lane & 15, side = (i >> 2) & 1;
    locate(g, min(p0 + (lane % PAIRS & ~15) + 15 * side, g.pairs - 1), &q, &ty, &n);
    img = (unsigned)(n - n0) * (unsigned)g.C * HW + plane0;
    const int y = 2 * ty - 1 + (i & 3), xx = side ? 4 * q + 4 : 4 * q - 1;
    edge_off = i < 8 && y >= 0 && y < g.H && xx >= 0 && xx < g.W
                   ? (img + (unsigned)y * (unsigned)g.W + (unsigned)xx) * 4u : kOutside;
  }

  __device__ __forceinline__ void issue(const PairGeo& g, int k, Pixels& px) const {
    const unsigned plane = (unsigned)g.H * (unsigned)g.W * 4u;
    int c = c_wave + 16 * k;
    unsigned add = 0;
    if constexpr (!FULL) {  // channels beyond C read the last plane; their bytes are masked
      const int own = min(c + group, g.C - 1);
      c = min(c, g.C - 1);
      add = (unsigned)(own - c) * plane;
    }
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(base + (size_t)c * plane), 0, g.reach, 0x00020000);
#pragma unroll
    for (int r = 0; r < 4; r++)
      px.own[r] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, own_off[r] + add, 0, 0));
    px.edge = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, edge_off + add, 0, 0));
  }

  // a DPP move; lanes without a source, and lanes outside the banks, keep old
  template <int CTRL, int BANKS>
  __device__ __forceinline__ static float dpp(float old, float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, 0xF,
                                                      BANKS, false));
  }

  // codes[s][e]: byte k of the lane's dword of position e of tile s
  __device__ __forceinline__ void quantize(const Pixels& px, const float (&qmn)[E], const float (&qinv)[E],
                                           float L, int k, unsigned (&codes)[2][E]) const {
    // the pixels beside the segment, for the first and the last lane of a group: row_shl:r brings
    // lane r's to lane 0, row_ror:11-r lane 4+r's to lane 15
    constexpr int kShl = 0x100, kShr = 0x110, kRor = 0x120, kLast = 0x8;
    const float e4[4] = {dpp<kRor + 11, kLast>(px.edge, px.edge),
                         dpp<kRor + 10, kLast>(dpp<kShl + 1, 0xF>(px.edge, px.edge), px.edge),
                         dpp<kRor + 9, kLast>(dpp<kShl + 2, 0xF>(px.edge, px.edge), px.edge),
                         dpp<kRor + 8, kLast>(dpp<kShl + 3, 0xF>(px.edge, px.edge), px.edge)};
    float t[4][4], te[4];  // B^T d of the four own columns and of the edge column
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const float col[4] = {px.own[0][c], px.own[1][c], px.own[2][c], px.own[3][c]};
      float o[4];
      Wino<2>::in1d(col, o);
#pragma unroll
      for (int i = 0; i < 4; i++) t[i][c] = o[i];
    }
    Wino<2>::in1d(e4, te);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      float l = dpp<kShr + 1, 0xF>(te[i], t[i][3]);  // the left neighbour's last column
      float r = dpp<kShl + 1, 0xF>(te[i], t[i][0]);  // the right neighbour's first column
      l = left_edge ? 0.0f : l;
      r = right_edge ? 0.0f : r;
      const float ra[4] = {l, t[i][0], t[i][1], t[i][2]}, rb[4] = {t[i][1], t[i][2], t[i][3], r};
      float v[2][4];
      Wino<2>::in1d(ra, v[0]);
      Wino<2>::in1d(rb, v[1]);
#pragma unroll
      for (int s = 0; s < 2; s++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const int e = 4 * i + j;
          // clamp(rne((x - min) * inv), 0, L): v_cvt_pk_u8_f32 rounds to nearest even and saturates
          // to [0, 255]; only the upper clamp of narrower codes needs an instruction
          float tq = (v[s][j] - qmn[e]) * qinv[e];
          if constexpr (!B8) tq = fminf(tq, L);
          codes[s][e] = __builtin_amdgcn_cvt_pk_u8_f32(tq, k, k == 0 ? 0u : codes[s][e]);
        }
    }
    // Pin this channel's arithmetic to its step: its results are first needed after the last
    // one, and left alone the compiler moves the arithmetic of all steps there, with the pixels
    // of all channels held in registers (or spilled) meanwhile.
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
      for (int e = 0; e < E; e++) asm volatile("" : "+v"(codes[s][e]));
    __builtin_amdgcn_sched_barrier(0);
  }

  // The lane's dwords into the code rows [E][kTiles][64 B] at ring.  d: the lane's dword of chunk `chunk`.
  __device__ __forceinline__ void store(const PairGeo& g, int chunk, int d, int lane, char* ring,
                                        const unsigned (&codes)[2][E]) const {
    const unsigned h = 1u << (g.bits - 1);
    const unsigned H8 = 0x80808080u, hh = h * 0x01010101u;
    unsigned mask = 0;  // bytes of channels that exist
#pragma unroll
    for (int b = 0; b < 4; b++)
      if (c_wave + 16 * b + group < g.C) mask |= 0xFFu << (8 * b);
#pragma unroll
    for (int s = 0; s < 2; s++) {
      const int row = PAIRS * s + lane % PAIRS;
      char* dst = ring + (unsigned)row * 64u + (unsigned)((chunk ^ row_swizzle_mfma32(row)) * 16) + 4u * (unsigned)d;
#pragma unroll
      for (int e = 0; e < E; e++) {
        const unsigned u = codes[s][e];
        // per-byte (code - h) mod 256 without borrows between bytes (h = 128: flip the top bit)
        unsigned v;
        if constexpr (B8)
          v = u ^ H8;
        else
          v = ((u | H8) - (hh & ~H8)) ^ ((u ^ ~hh) & H8);
        if constexpr (!FULL) v &= mask;
        *reinterpret_cast<unsigned*>(dst + e * (kTiles * 64)) = v;
      }
    }
  }
};

}  // namespace dev
}  // namespace lance
