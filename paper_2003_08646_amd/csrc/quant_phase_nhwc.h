// Transform + quantize of one block of TILES tiles x NBLK 64-channel blocks of F(2x2,3x3) into
// LDS from NHWC pixels: v^ = Q(B^T d B) (Algorithm 1; Eq. 7) formed in registers, the signed 8-bit
// codes written as code rows [NBLK][E][TILES][64 B] with the channels in their natural order (the
// order of the filter codes of an NHWC layer), the column sums of the unsigned codes left in LDS.
// The NHWC counterpart of quant_phase.h / quant_phase32.h, used by the one-kernel plans
// (conv_fused_c64.hip: 64 tiles x 1 block; conv_fused_c128.hip: 32 tiles x 2 blocks).
//
// Called by all 256 threads of a workgroup.  16 * NBLK lanes per tile: lane j holds the channels
// 4j .. 4j+3 (one 16-byte load per pixel of the 4x4 window; C is a multiple of 4), a thread
// group takes four tiles one after the other; the window of the next tile is requested before
// the current one is transformed.  The lane's four codes of a position are one dword of the
// code row; the column sum is a 16-lane DPP sum (added to LDS with an atomic when a tile has
// two blocks).
//
// ROLL (tile rows of a multiple of four tiles, so that four consecutive tiles from a multiple of four on
// share a row): a thread group takes four consecutive tiles and keeps the two pixel columns that a tile
// shares with the next one: 40 loads for the four instead of 64, two tiles ahead in the same registers.
// (N64 128 -> 128 56x56: 114.7 -> 109.6 us, N16 64 -> 64 224x224 212 -> 203, N128 64 -> 64 32x32 37.2 -> 36.7, N500
// 64 -> 64 8x8 20.5 -> 20.6.)
//
// LDS code rows are 64 bytes; the 16-byte chunk c of row p is stored at chunk c ^ row_swizzle(p)
// (what the fragment reads of the product phase expect).
#pragma once
#include "lance_device.h"
#include "nhwc_window.h"
#include "quant_phase.h"

namespace lance {
namespace dev {

// B8: 8-bit codes.  p0: first tile of the block.  ring: [NBLK][16][TILES][64 B].  cs_s:
// [16][TILES] int: every entry written here (NBLK = 1), or added to (NBLK = 2: zeroed by the caller
// before a barrier inside mid()).  mid(): run once after the first loads have been requested (all
// threads; may use barriers).  qp(e, &mn, &inv): the Eq. 7 parameters of position e, valid
// after mid().  Uses g.x as [N][H][W][C] (16-byte aligned), g.reach = its size in bytes.
template <bool B8, int TILES, int NBLK, bool ROLL, class Mid, class Qp>
__device__ __forceinline__ void quantize_block_nhwc_to_lds(const QuantBlockGeo& g, int p0,
                                                           char* ring, int* cs_s, int tid,
                                                           Mid&& mid, Qp&& qp) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  constexpr int M = 2, A = 4, E = 16;
  constexpr int kLanes = 16 * NBLK, kGroups = 256 / kLanes, kItems = TILES / kGroups;
  static_assert(kItems * kGroups == TILES, "tiles split evenly over the thread groups");
  constexpr unsigned kPlane = TILES * 64u, kBlock = E * kPlane;
  const int j = tid % kLanes, grp = tid / kLanes;
  const int jj = j & 15, blk = j >> 4;  // dword of the code row, channel block
  const bool lane_real = 4 * j < g.C;            // C is a multiple of 4: all four or none
  const int c0 = min(4 * j, g.C - 4);            // a real quad for the loads of padding lanes
  auto load = [&](int it, f4 (&w)[A * A]) {
    const int pt = min(p0 + kGroups * it + grp, g.P - 1);
    const int tx = pt % g.tw, t2 = pt / g.tw;
    const int ty = t2 % g.th, n = t2 / g.th;
    load_window_nhwc<M>(g.x, g.reach, n, ty * M - g.pad, tx * M - g.pad, c0, g.H, g.W, g.C, w);
  };
  // ROLL: columns 2i and 2i + 1 of the four tiles' common window, rows * 2 pixels
  constexpr int kHalves = kItems + 1, kHalvesAhead = 3;
  f4 half[ROLL ? kHalves : 1][A * 2];
  unsigned rowoff[A];
  bool rok[A];
  int x0 = 0;
  if constexpr (ROLL) {
    static_assert(kItems == 4, "four consecutive tiles per thread group");
    const int pt = min(p0 + kItems * grp, g.P - kItems);  // (P is a multiple of four)
    const int tx = pt % g.tw, t2 = pt / g.tw;
    const int ty = t2 % g.th, n = t2 / g.th;
    x0 = tx * M - g.pad;
#pragma unroll
    for (int r = 0; r < A; r++) {
      const int gy = ty * M - g.pad + r;
      rok[r] = gy >= 0 && gy < g.H;
      rowoff[r] = ((unsigned)n * (unsigned)g.H + (unsigned)gy) * (unsigned)g.W * ((unsigned)g.C * 4u);
    }
  }
  auto load_half = [&](int i, f4 (&w)[A * 2]) {
    unsigned coloff[2];
    bool cok[2];
#pragma unroll
    for (int s = 0; s < 2; s++) {
      const int gx = x0 + 2 * i + s;
      cok[s] = gx >= 0 && gx < g.W;
      coloff[s] = (unsigned)gx * ((unsigned)g.C * 4u) + (unsigned)c0 * 4u;
    }
#pragma unroll
    for (int r = 0; r < A; r++) {
      f4 row[2];
      load_row_nhwc<2>(g.x, g.reach, rowoff[r], rok[r], coloff, cok, row);
      w[2 * r] = row[0];
      w[2 * r + 1] = row[1];
    }
  };
  f4 win[ROLL ? 1 : 2][A * A];
  if constexpr (ROLL) {
#pragma unroll
    for (int i = 0; i < kHalvesAhead; i++) load_half(i, half[i]);
  } else {
    load(0, win[0]);
  }

  mid();
  __syncthreads();  // mid() may still read scratch inside the ring after its last barrier

  // Eq. 7 parameters as wave-uniform scalars
  float qmn[E], qinv[E];
#pragma unroll
  for (int e = 0; e < E; e++) {
    float mn, inv;
    qp(e, &mn, &inv);
    qmn[e] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(mn)));
    qinv[e] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(inv)));
  }
  const float L = (float)((1 << g.bits) - 1);
  const unsigned h = 1u << (g.bits - 1);
  const unsigned H8 = 0x80808080u, hh = h * 0x01010101u;
  const unsigned realmask = lane_real ? 0xFFFFFFFFu : 0u;

#pragma unroll
  for (int it = 0; it < kItems; it++) {
    if constexpr (ROLL) {
      if (it + kHalvesAhead < kHalves) load_half(it + kHalvesAhead, half[it + kHalvesAhead]);
    } else {
      if (it + 1 < kItems) load(it + 1, win[(it + 1) & 1]);
    }
    const int t = ROLL ? kItems * grp + it : kGroups * it + grp;  // code row of this item
    unsigned pk[E];               // unsigned codes of Eq. 7, byte i = channel 4j + i
#pragma unroll
    for (int e = 0; e < E; e++) pk[e] = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      float d[A][A];
#pragma unroll
      for (int r = 0; r < A; r++)
#pragma unroll
        for (int s = 0; s < A; s++) {
          if constexpr (ROLL) d[r][s] = half[it + s / 2][2 * r + s % 2][i];
          else d[r][s] = win[it & 1][r * A + s][i];
        }
      input_tile_transform<M>(d);
#pragma unroll
      for (int e = 0; e < E; e++) {
        // clamp(rne((x - min) * inv), 0, L): v_cvt_pk_u8_f32 rounds to nearest even and
        // saturates to [0, 255]; only the upper clamp of narrower codes needs an instruction
        float tq = (d[e / A][e % A] - qmn[e]) * qinv[e];
        if constexpr (!B8) tq = fminf(tq, L);
        pk[e] = __builtin_amdgcn_cvt_pk_u8_f32(tq, i, pk[e]);
      }
    }
    char* row = ring + (unsigned)blk * kBlock + (unsigned)t * 64u +
                (unsigned)(((jj >> 2) ^ row_swizzle(t)) * 16 + (jj & 3) * 4);
#pragma unroll
    for (int e = 0; e < E; e++) {
      const unsigned u = pk[e] & realmask;
      const int tot = row16_sum((int)__builtin_amdgcn_sad_u8(u, 0u, 0u));
      // per-byte (code - h) mod 256 without borrows between bytes (h = 128: flip the top bit)
      unsigned v;
      if constexpr (B8)
        v = u ^ H8;
      else
        v = ((u | H8) - (hh & ~H8)) ^ ((u ^ ~hh) & H8);
      *reinterpret_cast<unsigned*>(row + e * kPlane) = v & realmask;
      if (jj == 0) {
        if constexpr (NBLK == 1) cs_s[e * TILES + t] = tot;
        else atomicAdd(&cs_s[e * TILES + t], tot);
      }
    }
    // keep this tile's arithmetic here: left alone the compiler interleaves all four tiles and
    // holds their windows at once
    __builtin_amdgcn_sched_barrier(0);
  }
}

}  // namespace dev
}  // namespace lance
