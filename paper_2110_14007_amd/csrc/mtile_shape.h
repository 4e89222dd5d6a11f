// Launch shapes of the register-list tile kernel (mtile.h), shared by the
// kernel's launcher and the planner.  dpad: padded row length; fold: the seed
// sits in the row's padding; r: list entries per lane (K' = 2r); pr: the
// pruned scan, whose rows of 16 elements take short stages (a box is a stage)
// and smaller workgroups (a workgroup stages what any of its waves needs).
#pragma once

namespace tod {
namespace mt {

// Least rows of a box of the pruned scan (one box test per 128 rows and wave).
constexpr int kUnitRows = 128;

// Waves per workgroup.
constexpr int tile_waves(int dpad, bool fold, int r, bool pr) {
  return fold && r <= 8 ? (pr ? 4 : 16) : (dpad == 64 && !fold && r == 16) ? 8 : 4;
}
// 32-row sub-tiles per stage: the stage pair, seeds and queues of a 4-wave
// workgroup stay under 80 KiB so that at least two workgroups share a CU.
constexpr int stage_subs_base(int dpad) {
  return dpad == 16 ? 8 : (dpad == 32 ? 4 : (dpad == 64 ? 2 : 1));
}
constexpr int stage_subs(int dpad, bool fold, int r, bool pr) {
  return pr && dpad == 16                   ? 4
         : fold && r <= 8                   ? 16
         : (dpad == 64 && !fold && r == 16) ? 4
                                            : stage_subs_base(dpad);
}
// Query columns per wave / 32: two groups sharing every A fragment for rows
// of 512 elements with lists of up to 32 entries, whose 32-step MFMA chains
// otherwise need one LDS fragment per MFMA; one otherwise.  The two groups'
// operands take all 256 AGPRs; 64-entry lists for two groups (128 VGPRs)
// then leave the compiler too few registers, and it spills part of the
// operand to scratch memory.
constexpr int query_groups(int dpad, bool fold, int r) {
  return dpad >= 512 && !fold && r <= 16 ? 2 : 1;
}

// Workgroups of the plain scan that a compute unit holds at once.
constexpr int tile_resident(int dpad, bool fold, int r) {
  return r >= 32 || tile_waves(dpad, fold, r, false) > 4 || query_groups(dpad, fold, r) > 1 ? 1
         : r <= 8 && (dpad == 16 || dpad == 64 || dpad == 128)                             ? 3
                                                                                           : 2;
}

}  // namespace mt
}  // namespace tod
