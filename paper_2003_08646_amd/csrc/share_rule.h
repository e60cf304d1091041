// How many waves of the small-channel kernel (conv_fused_c16.hip) share 64 tiles.
#pragma once

namespace lance {

// Time of the kernel in us with `split` waves to 64 tiles: a fixed part, and for each workgroup of a compute unit (the
// second one adds to the first one's time, the vector ALUs are shared) the constants, the channels' transforms and
// the wave's products of 32 filters x 32 tiles.  Fitted on 110 layers of 5000 to 90000 tiles with caller's ranges, three
// splits each: 10 % off on average (NHWC 25 %).
inline double c16_us(long long tiles, int C, int K, bool nhwc, int split) {
  const long long wgs = ((tiles + 63) / 64 * split + 3) / 4, kt = (K + 31) / 32;
  const double load = (double)((wgs + 255) / 256) * 0.8;
  const double parts = (double)(split == 1 ? 2 * kt : split == 2 ? kt : (kt + 1) / 2);
  return nhwc ? -0.8 + (load > 1.0 ? load : 1.0) * (3.3 + 1.1 * C + 5.4 * parts)
              : 3.9 + (load > 1.0 ? load : 1.0) * (1.8 + 0.37 * C + 3.9 * parts);
}

// More than one where workgroups of 256 tiles leave compute units idle and the transform, which every wave repeats, is the
// smaller part.  Us per call with 1 / 2 / 4 (caller's ranges): N8 1->272 99^2 NHWC 74 / 45 / 41, N11 3->103 105^2 42 / 29 /
// 27, N128 16->16 32^2 18 / 15 / 17, N53 3->33 19x57 23 / 16 / 12, N16 3->64 224^2 55 / 58 / 70.
// Not where most compute units have work as it is (NHWC: half of them) and Y, which every split writes in smaller pieces,
// exceeds the last-level cache: N959 3->294 16^2 72 / 96 / 79, N803 16->209 20^2 84 / 93 / 102, N229 15->872 24^2 NHWC 236 with
// one, 280 with four.
inline int c16_split(long long tiles, int C, int K, bool nhwc, long long y_bytes) {
  if (tiles > (nhwc ? 128 : 205) * 256 && y_bytes > 256LL << 20) return 1;
  const double one = c16_us(tiles, C, K, nhwc, 1), two = c16_us(tiles, C, K, nhwc, 2), four = c16_us(tiles, C, K, nhwc, 4);
  // (of 200 other layers none lost more than 2 % with these margins)
  if ((nhwc ? 0.75 : 0.85) * one <= (two < four ? two : four)) return 1;
  return two <= four ? 2 : 4;
}

}  // namespace lance
