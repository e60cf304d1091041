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
  int C, H, W, Ho, Wo, pad, th, npr, pairs, bits;  // npr: pairs per tile row; pairs: of the whole batch
  int tiles;       // of the whole batch (pairs of any two tiles, where npr is the tiles per row)
  unsigned th_magic, npr_magic;
  int exact;       // fast_div is exact for every pair (false only for NHWC rows of very many pairs)
  unsigned reach;  // extent of the buffer descriptors: bytes from a plane of a block's first image
};

// Pair (or tile) p of the batch: pair q of tile row ty of image n.
template <bool NHWC>
__device__ __forceinline__ void locate_pair(const PairGeo& g, int p, int* q, int* ty, int* n) {
  const bool fast = !NHWC || g.exact;
  const int t2 = fast ? fast_div(p, g.npr_magic) : p / g.npr;
  *q = p - t2 * g.npr;
  *n = fast ? fast_div(t2, g.th_magic) : t2 / g.th;
  *ty = t2 - *n * g.th;
}

// Four stored codes from four unsigned ones: per byte (code - h) mod 256 without borrows between bytes
// (h = 128: flip the top bit).
template <bool B8>
__device__ __forceinline__ unsigned stored_codes(unsigned u, unsigned h) {
  const unsigned H8 = 0x80808080u, hh = h * 0x01010101u;
  if constexpr (B8) return u ^ H8;
  return ((u | H8) - (hh & ~H8)) ^ ((u ^ ~hh) & H8);
}

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

  // block: PAIRS consecutive pairs of the batch
  __device__ __forceinline__ void setup(const PairGeo& g, int block, int c_first, int lane) {
    const int p0 = block * PAIRS;
    c_wave = c_first;
    group = lane / PAIRS;
    const unsigned HW = (unsigned)g.H * (unsigned)g.W;
    const int n0 = fast_div(fast_div(p0, g.npr_magic), g.th_magic);
    base = reinterpret_cast<const char*>(g.x + (size_t)n0 * g.C * HW);
    int q, ty, n;
    locate_pair<false>(g, min(p0 + lane % PAIRS, g.pairs - 1), &q, &ty, &n);
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
    locate_pair<false>(g, min(p0 + (lane % PAIRS & ~15) + 15 * side, g.pairs - 1), &q, &ty, &n);
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
        unsigned v = stored_codes<B8>(codes[s][e], h);
        if constexpr (!FULL) v &= mask;
        *reinterpret_cast<unsigned*>(dst + e * (kTiles * 64)) = v;
      }
    }
  }
};

// The same from NHWC pixels, any padding and width, C a multiple of 4 and X 16-byte aligned: 16 lanes per
// pair and channel block, lane j holds the channels 4j .. 4j+3 (dword j of the code row, channels in
// their natural order).  The pair's window is six pixel columns of four 16-byte loads, taken column by
// column: a column goes through B^T d once for both tiles, and a position's four codes are a whole dword that
// goes to LDS at once, so no codes wait in registers.  Pixels outside the image have an offset beyond
// the buffer: one add per load and nothing after it.
// ANY: the pair is any two consecutive tiles of the batch, each with its own window of four columns (32 loads, eight
// column passes), so that no tile row ends in half a pair.
//
// Called by all 512 threads.  LDS rows and chunks as above.
template <bool B8, int PAIRS, bool ANY>
struct PairPhaseNhwc {
  typedef float f4 __attribute__((ext_vector_type(4)));
  static constexpr int E = 16, kTiles = 2 * PAIRS, kEarly = 4;
  static constexpr int kBuffers = 6;                          // pixel columns in flight or in use
  static constexpr int kWindows = ANY ? 2 : 1, kColumns = ANY ? 4 : 6;  // columns of a window
  static constexpr unsigned kOutside = 0xFFFFFFF0u;  // beyond any X (the whole of which is one buffer)

  unsigned rowoff[kWindows][4], coloff[kWindows][kColumns];  // rows that do not exist have kOutside
  bool cok[kWindows][kColumns];
  char* dst;         // the lane's dword of position 0 of the left tile
  unsigned mask;     // all ones where the lane's channels exist

  // block: PAIRS consecutive pairs of the batch; pair: the lane's among them; cblk: channel block;
  // ring: its code planes [E][kTiles][64 B]
  __device__ __forceinline__ void setup(const PairGeo& g, int block, int pair, int cblk, int lane, char* ring) {
    const int p0 = block * PAIRS;
    const unsigned px = (unsigned)g.C * 4u, row_bytes = (unsigned)g.W * px;
    const int j = lane & 15, c = 64 * cblk + 4 * j;
    mask = c < g.C ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int w = 0; w < kWindows; w++) {
      int q, ty, n;
      locate_pair<true>(g, ANY ? min(2 * (p0 + pair) + w, g.tiles - 1) : min(p0 + pair, g.pairs - 1), &q, &ty, &n);
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int y = 2 * ty - g.pad + r;
        rowoff[w][r] = y >= 0 && y < g.H ? ((unsigned)n * (unsigned)g.H + (unsigned)y) * row_bytes : kOutside;
      }
#pragma unroll
      for (int s = 0; s < kColumns; s++) {
        const int x = (ANY ? 2 : 4) * q - g.pad + s;
        cok[w][s] = x >= 0 && x < g.W;
        coloff[w][s] = (unsigned)x * px + (unsigned)min(c, g.C - 4) * 4u;
      }
    }
    dst = ring + (unsigned)pair * 64u + (unsigned)(((j >> 2) ^ row_swizzle_mfma32(pair)) * 16 + 4 * (j & 3));
  }

  // pixel column s of the pair (ANY: 0 .. 3 of the first tile, 4 .. 7 of the second)
  __device__ __forceinline__ void issue(const PairGeo& g, int s, f4 (&w)[4]) const {
    const int win = s / kColumns, i = s % kColumns;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g.x), 0, g.reach, 0x00020000);
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const unsigned off = cok[win][i] && rowoff[win][r] != kOutside ? rowoff[win][r] + coloff[win][i] : kOutside;
      w[r] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
    }
  }

  // B^T d of one pixel column, in place
  __device__ __forceinline__ static void column(f4 (&w)[4]) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const float d[4] = {w[0][q], w[1][q], w[2][q], w[3][q]};
      float t[4];
      Wino<2>::in1d(d, t);
#pragma unroll
      for (int i = 0; i < 4; i++) w[i][q] = t[i];
    }
  }

  // The codes of position column j of tile s (0 left, 1 right): a + b or a - b of two pixel columns.
  template <bool SUM>
  __device__ __forceinline__ void codes(const PairGeo& g, int s, int j, const f4 (&a)[4], const f4 (&b)[4],
                                        const float (&qmn)[E], const float (&qinv)[E]) const {
    static_assert(PAIRS % 16 == 0, "both tiles of a pair have the same swizzle");
    const float L = (float)((1 << g.bits) - 1);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int e = 4 * i + j;
      unsigned u = 0;
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const float v = SUM ? a[i][q] + b[i][q] : a[i][q] - b[i][q];
        float tq = (v - qmn[e]) * qinv[e];  // Eq. 7 as in PairPhase
        if constexpr (!B8) tq = fminf(tq, L);
        u = __builtin_amdgcn_cvt_pk_u8_f32(tq, q, u);
      }
      *reinterpret_cast<unsigned*>(dst + (unsigned)(PAIRS * s * 64 + e * kTiles * 64)) =
          stored_codes<B8>(u, 1u << (g.bits - 1)) & mask;
    }
  }
  // All codes of the pair.  w: the first kEarly pixel columns, requested.  late(): requests what the caller
  // needs next, when half of the columns' registers are free.
  template <class Late>
  __device__ __forceinline__ void run(const PairGeo& g, f4 (&w)[kBuffers][4], const float (&qmn)[E],
                                      const float (&qinv)[E], Late&& late) const {
    if constexpr (ANY) {
      issue(g, 4, w[4]);
#pragma unroll
      for (int s = 0; s < 3; s++) column(w[s]);
      codes<false>(g, 0, 0, w[0], w[2], qmn, qinv);
      codes<true>(g, 0, 1, w[1], w[2], qmn, qinv);
      codes<false>(g, 0, 2, w[2], w[1], qmn, qinv);
      __builtin_amdgcn_sched_barrier(0);
      issue(g, 5, w[5]);
      issue(g, 6, w[0]);
      column(w[3]);
      codes<false>(g, 0, 3, w[1], w[3], qmn, qinv);
      __builtin_amdgcn_sched_barrier(0);
      issue(g, 7, w[2]);
      column(w[4]);
      column(w[5]);
      column(w[0]);
      codes<false>(g, 1, 0, w[4], w[0], qmn, qinv);
      __builtin_amdgcn_sched_barrier(0);
      late();
      codes<true>(g, 1, 1, w[5], w[0], qmn, qinv);
      codes<false>(g, 1, 2, w[0], w[5], qmn, qinv);
      column(w[2]);
      codes<false>(g, 1, 3, w[5], w[2], qmn, qinv);
      return;
    }
    issue(g, 4, w[4]);
#pragma unroll
    for (int s = 0; s < 3; s++) column(w[s]);
    codes<false>(g, 0, 0, w[0], w[2], qmn, qinv);
    codes<true>(g, 0, 1, w[1], w[2], qmn, qinv);
    codes<false>(g, 0, 2, w[2], w[1], qmn, qinv);
    column(w[3]);
    codes<false>(g, 0, 3, w[1], w[3], qmn, qinv);
    __builtin_amdgcn_sched_barrier(0);
    issue(g, 5, w[5]);
    column(w[4]);
    codes<false>(g, 1, 0, w[2], w[4], qmn, qinv);
    __builtin_amdgcn_sched_barrier(0);
    late();
    codes<true>(g, 1, 1, w[3], w[4], qmn, qinv);
    codes<false>(g, 1, 2, w[4], w[3], qmn, qinv);
    column(w[5]);
    codes<false>(g, 1, 3, w[3], w[5], qmn, qinv);
  }
};

}  // namespace dev
}  // namespace lance
