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

// Whether the sweep's waves raise their priorities through a group (stage kernel).  They gain in one
// round and in many.  Where a second or third round leaves a wave slot of every SIMD idle, the waves
// that have one more group are on the critical path, and the priorities let those that are finishing
// pass them (steps, raised against not, per cent): 2 waves per SIMD, 1 to 1.5 rounds: fp16 P3 -5,
// FP64 P2 -6, FP32 P3 -2, FP32 P1 adjoint -7; 2 to 2.5: fp16 -2..-8, FP64 and FP32 0..-4; 3 to 3.5:
// fp16 P2 -4..-1, FP32 +1; 1.5 to 2, 2.5 to 3, 3.5 on: +2..+9.  3 per SIMD, 1 to 1.33 rounds: FP64 P1
// -7, FP32 P1 -5; 1.33 to 1.67: -3..0; beyond +3..+9.
//   blocks: workgroups launched (sweep_blocks), per_cu: those that fit a CU (waves per SIMD),
//   rounds: from this many full rounds on a partial one no longer matters (mixed modes 4, others 3)
inline bool rising_priority(int64_t ngroups, int64_t blocks, int per_cu, int64_t rounds) {
  const int64_t waves = 4 * blocks, full = ngroups / waves, rest = ngroups % waves;
  return full == 0 || full >= rounds || rest == 0 || rest * per_cu > waves * (per_cu - 1);
}

}  // namespace tetdg
