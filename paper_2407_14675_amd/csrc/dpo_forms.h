// Choice between the direct sweeps' two forms (host).
#pragma once

namespace dpo {

constexpr int kChipNodes = 5 * 64 * 1024;  // nodes in flight at five waves per SIMD

// Which form a direct sweep takes.  The cell cache saves an evaluation its
// look-up and costs more than one where a foot leaves the cell: it pays where the
// table is long for the number of cell changes, which grows with the thrust step
// (reach: the longest, in cells).  Cell cache / keyed corners, us:
//   crown, Heun, 110 x 30^3: reach 0.007, 24 entries 181 / 214, 72 395 / 542; 0.03, 24
//     230 / 223, 36 281 / 305; 0.07, 48 437 / 406, 72 540 / 568
//   orbit, Heun, 110 x 30^3: 0.016, 24 entries 218 / 212, 48 348 / 366; 0.05, 48 401 /
//     381, 72 525 / 536; 0.1, 72 612 / 559
//   orbit, Euler, 110 x 30^3: 0.018, 24 entries 168 / 173; 0.05, 36 269 / 249, 72 399 /
//     423; 0.1, 72 474 / 446
//   eikonal, 256^2, steps of a cell: 72 entries 95 / 56
// The Heun foot's golden section does not pay for it, whose cell-cache form spills 20
// registers and more (orbit, 60 x 25^3, scan 64 + golden 12 233 / 210); the Euler foot's
// does for a shorter reach (crown, 110 x 30^3: 330 / 422 at 0.007, 395 / 434 at 0.03,
// 516 / 458 at 0.07).  Nor do a walk's few evaluations, but for the crown's Euler foot
// below one load of the chip (12^4 8.0 / 9.3, 40 x 20^3 14.7 / 15.8, 110 x 30^3 66.6 / 64.5;
// orbit, 110 x 30^3 81 / 72).  Sweeps that leave the chip partly idle wait for each look-up with
// little beside them: the Heun foot below one load of the chip (25 x 15^3, 72 entries: 63
// / 51), the orbit model with the Euler foot below half of one (12^4, scan 64 + golden
// 12: 42 / 39).
// mode: 0 table, 1 scan + golden, 2 seeded, 3 table walk; entries of the table; free nodes.
inline bool keep_cells(int mode, bool crown, bool heun, int entries, int nodes, float reach) {
  const bool scan = mode == 1 || mode == 2;
  if (!((scan ? 5 * entries / 8 : entries) >= 16.0f + 800.0f * reach)) return false;
  if (mode == 3) return crown && !heun && nodes < kChipNodes;
  if (heun) return !scan && nodes >= kChipNodes;
  return crown || nodes >= kChipNodes / 2;
}

}  // namespace dpo
