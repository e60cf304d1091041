// Host side of conv_fused_pos.h and its F(2x2,3x3) instances.
#include "conv_fused_pos.h"

namespace lance {
namespace pos {
hipError_t launch_m4(const CpArgs& a, bool clamp, int cpl, int load, int kg, hipStream_t s);

// How a layer is cut into workgroups: 16 tiles x 16*kg filters, nw waves each.
struct Shape {
  int kg, nw, nky;
  long long groups;
  double cost;  // rounds x relative time of a workgroup
};

// The shape with the smallest (rounds of resident workgroups) x (relative time of a workgroup).  A
// compute unit holds one workgroup of 16 (m = 4: 12) waves, or two of eight, which then share its
// units but overlap their phases.  Relative times from sweeps over layers of 3 to 512 channels: a
// workgroup of 16 waves takes 1.08x and 1.25x as long with twice and four times the filters, two of
// eight waves side by side 1.3x .. 1.6x (64 channels, 64 filters, 784 blocks of tiles: 36 us with 16
// waves, 27 us with eight; 61 filters, 135 blocks: 15.5 and 15.9 us); m = 4: 1.12x and 1.45x.
static Shape shape_of(const Geo& g) {
  const long long tb = (g.P + 15) / 16;
  Shape best{1, 16, 0, 0, 0.0};
  auto consider = [&](int nw, int kg, int slots, double cost) {
    const int nky = (g.K + 16 * kg - 1) / (16 * kg);
    const double c = (double)((tb * nky + slots - 1) / slots) * cost;
    if (best.nky == 0 || c < best.cost) best = Shape{kg, nw, nky, tb * nky, c};
  };
  constexpr double kCost16[3] = {1.0, 1.08, 1.25}, kCost8[3] = {1.3, 1.4, 1.6}, kCost12[3] = {1.0, 1.12, 1.45};
  for (int i = 0; i < 3; i++) {
    consider(g.m == 2 ? 16 : 12, 1 << i, 256, g.m == 2 ? kCost16[i] : kCost12[i]);
    // (two workgroups of eight waves need half of the LDS each)
    if (g.m == 2 && g.NB <= 4) consider(8, 1 << i, 512, kCost8[i]);
  }
  return best;
}
}  // namespace pos

static bool conv_fused_pos_applicable(const Geo& g) {
  return (long long)g.N * g.C * g.H * g.W * 4 < 0x7FF00000LL &&
         (long long)g.N * g.K * g.Ho * g.Wo * 4 < 0xFFFFFFF0LL &&
         g.NB <= (g.m == 2 ? pos::most_blocks<2>() : pos::most_blocks<4>());
}

// Where the line lies (us per fused call, the plan that would run otherwise against this one; N, C,
// K, image):
//  * F(4x4), at most 16 channels: always (the fallback plan: N14 16->32 116x130 124 -> 41,
//    N9 16->128 97^2 NHWC 194 -> 111, N5 16->512 12^2 123 -> 16; N62 4->68 213x224 1474 -> 1082).
//  * F(2x2), at most 16 channels: up to 12800 tiles, and not where conv_fused_c16 with several waves to 64
//    tiles is estimated to take less than 0.85 of this plan's time, 1.2 us + 3.9 us per round (17 % off on 75 layers of
//    4000 to 12800 tiles), with dynamic ranges counting its reduction kernel.  This plan / that one, caller's ranges: N1
//    3->64 224^2 15.7 / 10.6, 7->68 with 12540 tiles 25.8 / 16.8, 2->40 with 8658 12.9 / 9.9, 5->50 with 5780 9.0 / 12.1, 16->61
//    with 11913 14.9 / 19.0; dynamic: N1 3->64 224^2 22.2 / 19.3, and little with more than 256 filters (2->371 with 7752 tiles
//    51.2 / 48.2, 16->290 with 7605 44.5 / 44.7), which stay here.  NHWC layers too (9->430 with 7569 tiles 45.7 / 70.6).
//  * F(2x2), 17 to 128 channels: up to two workgroups of eight waves per compute unit (N4 32->128 63^2
//    31.5 -> 21, N1 64->128 112^2 18.9 -> 14.4); one per compute unit where conv_fused_pairs.hip takes the
//    layer in one block of filters (caller's ranges, this plan / that one: N1 128->128 112^2 17.9 / 11.3, N16
//    128->128 28^2 17.2 / 12.2, N10 64->64 56^2 14.9 / 10.8; at 256 workgroups they meet: N4 64->64 56^2 9.7 /
//    9.9, N8 128->128 28^2 11.1 / 11.6; with two blocks of filters N20 48->96 28^2 13.4 / 14.1).  Not with one
//    channel block and at most 16 filters, of which that kernel computes 64: N20 56->8 109x8 8.6 / 9.7, N12
//    17->12 112x20 9.0 / 9.8, N15 64->5 169x8 8.6 / 9.4 (dynamic ranges 15.0 / 15.7 at most); 17 to 21 filters
//    9.8 / 9.8, two channel blocks from 5 filters on 12.5 / 10.5.
//    NHWC, 1258 layers between one and two workgroups per compute unit, the median of this plan's time over that one's for
//    17..32 / 33..64 / 65..128 / 129..192 / 257..399 filters, with caller's ranges: one channel block 0.97 / 1.12 / 0.84 / 0.69 /
//    0.49, two blocks 1.12 / 1.25 / 1.29 / 0.92 / 0.71 (dynamic ranges 0.05 to 0.1 more): in one block of filters
//    there too, from 17 or 33 filters on.  Where four filters are not one store (one block 0.83 / 0.87 / 0.62 / ..., two
//    1.03 / 1.10 / 1.08 / 0.73 / 0.49) two blocks only, with caller's ranges 33 to 72 filters (73..128: 0.83 to 1.24).
//    Two blocks and dynamic ranges: from one filter on (1.07 and 1.10 up to 16), where that kernel takes pairs of a
//    tile row (of any two tiles: 0.89 to 0.96).  With several blocks of filters
//    few workgroups do all the work: N2 64->704 28^2 15.9 / 51.2 us, N1 100->3218 15x24 19.1 / 68.0.
//  * the rest: one workgroup per compute unit (N1 512->512 28^2 23 -> 16.7, N1 128->256 56^2 F(4x4)
//    44 -> 15, N4 256->512 28^2 24 against 28, N23 38->52 108^2 F(4x4) 51 against 95).
static bool nhwc_pairs_preferred(const Geo& g) {
  if (!conv_fused_pairs_nhwc_applicable(g) || g.K > 64 * g.NB) return false;
  const bool is_static = (g.flags & LANCE_INPUT_RANGE_STATIC) != 0, whole = g.K % 4 == 0;
  if (g.NB == 1) return whole && g.K > (is_static ? 32 : 16);
  if (conv_fused_any_pairs(g)) return whole && g.K > 16;
  return !is_static || (whole ? g.K > 16 : g.K > 32 && g.K <= 72);
}

bool conv_fused_pos_preferred(const Geo& g, bool x_aligned) {
  if (!conv_fused_pos_applicable(g)) return false;
  if (g.C <= 16) {
    if (g.m == 4) return true;
    if (g.P > 12800) return false;
    const bool is_static = (g.flags & LANCE_INPUT_RANGE_STATIC) != 0;
    if (is_nhwc(g) || !conv_fused_c16_applicable(g) || (!is_static && g.K > 256)) return true;
    return conv_fused_c16_us(g) + (is_static ? 0.0 : 5.0) >= 0.85 * (1.2 + 3.9 * pos::shape_of(g).cost);
  }
  const bool pairs = is_nhwc(g) ? x_aligned && nhwc_pairs_preferred(g)
                                : conv_fused_pairs_applicable(g) && g.K <= 64 * g.NB && (g.NB == 2 || g.K > 16);
  const bool two = g.m == 2 && g.NB <= 2 && !pairs;
  return pos::shape_of(g).groups <= (two ? 512 : 256);
}

// Whether every workgroup reduces the records of the range pass for itself, or a reduction kernel does
// it once (3 to 4 us).  A compute unit's workgroups of one round after the other each read the records
// in batches of eight per thread, about 0.5 us a batch.  Over 1200 layers of both tile sizes the two
// meet at 8 batches: at 10 to 14 the workgroups' own reduction costs 0.5 to 5 us more (N88 3->12 72x57
// F(4x4) 60.0 -> 55.3 us per call with the kernel), on large first layers up to half of the call (N203
// 1->128 123x123 F(4x4) 2024 -> 1272 us); below 4 the kernel costs 2 to 4.6 us more.
bool conv_fused_pos_can_merge(const Geo& g, int count) {
  const pos::Shape sh = pos::shape_of(g);
  const long long slots = sh.nw == 8 ? 512 : 256, groups = sh.nw * 64 / (2 * g.E);
  return (sh.groups + slots - 1) / slots * ((count + 8 * groups - 1) / (8 * groups)) <= 8;
}

hipError_t launch_conv_fused_pos(const Geo& g, const float* x, const int8_t* uq,
                                 const float* u_range, const int32_t* u_rowsum,
                                 const float* partial, int count, int merge, float* v_range, float* y,
                                 hipStream_t s) {
  if (!conv_fused_pos_applicable(g)) return hipErrorInvalidValue;
  const bool is_static = (g.flags & LANCE_INPUT_RANGE_STATIC) != 0 || !merge;
  const pos::Shape sh = pos::shape_of(g);
  if (sh.groups > 0x7FFFFFFFLL) return hipErrorInvalidValue;
  const pos::CpArgs a{x, uq, u_range, u_rowsum, partial, v_range, y, nullptr, count,
                      (g.flags & LANCE_RANGE_PER_TENSOR) ? 1 : 0, is_static ? 1 : 0,
                      g.N, g.C, g.H, g.W, g.K, g.pad, g.P, g.th, g.tw, g.Ho, g.Wo, g.bits, g.bits_w,
                      g.NB, g.Q, g.CB == 16 ? 1 : (is_packed(g) ? 2 : 0), sh.nky,
                      (unsigned)((size_t)g.N * g.C * g.H * g.W * 4),
                      (unsigned)((size_t)g.N * g.K * g.Ho * g.Wo * 4), 0};
  // One channel per lane where four would leave waves without work (at most two blocks), and where
  // NHWC pixels cannot be loaded four channels at a time.
  int load, cpl = g.NB > 2 ? 4 : 1;
  if (is_nhwc(g)) {
    const bool wide = g.m == 2 && cpl == 4 && g.C % 4 == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    load = wide ? pos::kNhwc4 : pos::kNhwc1;
    if (!wide) cpl = 1;
  } else {
    load = patch_edge_cols_only(g) ? pos::kRowsEdge : pos::kRowsAny;
  }
  // 8-bit codes saturate in the conversion; ranges of the same tensor are exceeded by no number, but an
  // undefined value (which ranges skip) takes the last code here as in every other plan
  const bool clamp = g.bits < 8;
  if (g.m == 4) return pos::launch_m4(a, clamp, cpl, load, sh.kg, s);
  if (sh.nw == 16)
    return clamp ? pos::launch<2, 16, true>(a, cpl, load, sh.kg, s) : pos::launch<2, 16, false>(a, cpl, load, sh.kg, s);
  return clamp ? pos::launch<2, 8, true>(a, cpl, load, sh.kg, s) : pos::launch<2, 8, false>(a, cpl, load, sh.kg, s);
}

}  // namespace lance
