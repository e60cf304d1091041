// The F(4x4,3x3) instances of conv_fused_pos.h.
#include "conv_fused_pos.h"

namespace lance {
namespace pos {

hipError_t launch_m4(const CpArgs& a, bool clamp, int cpl, int load, int kg, hipStream_t s) {
  return clamp ? launch<4, 12, true>(a, cpl, load, kg, s) : launch<4, 12, false>(a, cpl, load, kg, s);
}

}  // namespace pos
}  // namespace lance
