// Items of the workgroups of a kernel that walks n items (at least one to a workgroup) with a stride.  Workgroups
// are dealt to the 8 accelerator dies (XCDs, each with its own L2) round robin by their index.  Every die gets a contiguous
// range, so that neighbouring items share an L2, as long as its number of workgroups, and deals it to them, so that
// a last, partial round is spread over all dies.  (With xcd_contiguous() as first item and the grid as stride the last
// round runs on the first dies alone: NHWC range passes of 1 to 1.5 rounds took 16 % longer than without any order.)
#pragma once
#include "lance_device.h"

namespace lance {
namespace dev {

// each, rest: n / blocks and n % blocks, and magic = div_magic(blocks) from the host: two divisions by a variable here
// took 0.2 us.  At most 1024 workgroups (the products below).
struct XcdRange {
  int first, end, step;
  __device__ __forceinline__ XcdRange(int each, int rest, unsigned magic, int block, int blocks) {
    constexpr int kXcd = 8;
    const int x = block % kXcd, q = blocks / kXcd, r = blocks % kXcd;
    const int mine = q + (x < r ? 1 : 0), before = x * q + (x < r ? x : r);
    first = each * before + fast_div(rest * before, magic) + block / kXcd;
    end = each * (before + mine) + fast_div(rest * (before + mine), magic);
    step = mine;
  }
};

}  // namespace dev
}  // namespace lance
