// Launch arithmetic of the kernels whose wavefronts sweep 16-element groups (host only, no HIP).
#pragma once
#include <cstdint>

namespace tetdg {

// Workgroups of four wavefronts for ngroups groups, of which `fill` fit the device at once: one group
// per wavefront where they fit.  From 8 on the count is a multiple of 8 (the same share of the
// groups for every XCD), rounded up unless that passes `fill`: rounded down, a few groups wait for
// a second round (FP32 P2 step, 3060 groups, 768 workgroups fit: 760 took 162 us, 768 take 129).
inline int64_t sweep_blocks(int64_t ngroups, int64_t fill) {
  if (fill < 1) fill = 1;
  int64_t n = (ngroups + 3) / 4;
  if (n >= 8) n = (n + 7) / 8 * 8;
  if (n > fill) n = fill >= 8 ? fill / 8 * 8 : fill;
  return n < 1 ? 1 : n;
}

}  // namespace tetdg
