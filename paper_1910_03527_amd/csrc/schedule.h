// Work-unit lengths of the sigma contraction: host rules without device code.
#pragma once
#include <algorithm>
#include <cstdint>

namespace mbefci {

constexpr int kCus = 256;

// Tile width where nothing is tuned (calls of one sigma, one CASCI per launch
// sequence).  10 orbitals, contraction in us with 32, 64 and 128: one CASCI of
// 252 x 252 strings 15.2, 11.4, 11.5, of 45 x 252 12.4, 9.6, 9.6, 24 of 252 x
// 252 159, 129, 150 (two waves per string hold eight column blocks each and
// leave one wave per SIMD).  9 orbitals, 126 x 126: one 8.5 and 7.8, 24 34.8 and
// 35.6 with 32 and 64; 8 orbitals, 70 x 70: one 6.8 and 6.6, 300 83 and 114.
inline int default_tile(int n) { return n > 10 ? 32 : 64; }

// Up to kStringMax orbitals a unit is a number of steps, each of the alpha
// strings that a workgroup takes at a time (string_spw).  The most steps that
// leave a plan with `steps` of them in all four units per CU.
inline int string_unit_limit(int64_t steps) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(steps / (4 * kCus), INT32_MAX));
}
// Steps per unit: the tuned number (0: 16), at most the limit.
inline int string_unit_steps(int tuned, int64_t steps) {
  return std::min(tuned > 0 ? tuned : 16, string_unit_limit(steps));
}

// The tuner times 4, 8, 16 and 32 steps per unit as far as the plan's limit
// tells them apart, and keeps one schedule per active size for every later
// plan.  A best length at a limit below 32 says nothing of longer ones: it is
// kept as -limit, and a plan with a higher limit (and more than the one length
// to choose from) is timed anew.
inline int schedule_kept(int best, int limit) {
  return limit < 32 && best >= limit ? -limit : best;
}
inline bool schedule_covers(int kept, int limit) {
  return kept > 0 || limit <= std::max(4, -kept);
}
inline int schedule_steps(int kept) { return kept > 0 ? kept : std::max(16, -kept); }

// Above kStringMax orbitals a unit is a number of tiles: the tuned one, or (0)
// 16, or 8 where the busiest CU then takes fewer tiles in all.  Units are
// dealt to the CUs, and the last, partly filled turn costs as much as a full
// one (a unit's set-up decides between equals).  units(l): units of l tiles.
// Contraction in us with 8 and 16: 12 orbitals, 792 x 495 strings (56 tiles on
// a CU against 64) 184 and 197, 495 x 495 (32, 32) 108 and 104; 11 orbitals,
// 462 x 330 (24, 32) 77 and 89, 462 x 462 (32, 32) 93 and 89; 13 orbitals,
// 1,716 x 13 (8, 16) 44 and 72, 1,287 x 78 (16, 16) 87 and 77; 14 orbitals,
// 3,003 x 91 (40, 48) 238 and 250.
template <class Units>
inline int pair_unit_tiles(int tuned, Units&& units) {
  if (tuned > 0) return tuned;
  auto busiest = [&](int l) { return ((int64_t)units(l) + kCus - 1) / kCus * l; };
  return busiest(8) < busiest(16) ? 8 : 16;
}

}  // namespace mbefci
