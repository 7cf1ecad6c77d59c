// form_limits.hpp -- largest batch, by component count, that a call leaving the
// launch shape to the library (grid, block and the lanes options 0) runs with a
// team of lanes per mixture, and with a lane pair per mixture in one launch (the
// fused form).  Row 0: the flash; row 1: the stability analysis alone.  0: never.
// autotune.py and the tests read these tables.
#pragma once

#include <stdint.h>

namespace ptf {

// Teams.  A team takes 8 (nc <= 4) or 16 lanes where the lane pair takes two, so it
// wins while the device has lanes to spare.  Measured (MI355X, us per call, team /
// lane pair):
//   flash: nc 3 168 / 247 at 2000 mixtures, 248 / 314 at 16,000, 305 / 272 at
//   24,000; nc 4 352 / 351 at 20,000; nc 5 254 / 383 at 4000, 378 / 393 at 8000, 473 / 433
//   at 12,000; nc 8 269 / 463 at 1000, 481 / 557 at 10,000, 620 / 629 at 12,000; nc 10
//   607 / 650 at 10,000; nc 12 (own sets) 893 / 1186 at 4000, 1247 / 1452 at 10,000,
//   1510 / 1203 at 12,000.
//   The stability analysis has less for a team to share (the substitution of a trial
//   is the same in all its lanes), so it wins only while every SIMD holds one
//   wavefront (8 or 4 mixtures each, 1024 SIMDs): nc 3 90 / 112 at 8000, 139 / 133 at
//   19,000; nc 5 98 / 142 at 4000, 163 / 142 at 8000; nc 8 153 / 213 at 4000, 223 / 204 at
//   8000; nc 12 235 / 300 at 4000, 344 / 300 at 9000.
constexpr int64_t kTeamMaxN[2][21] = {
    {0, 0, 20000, 20000, 20000, 10000, 10000, 10000, 10000, 10000, 10000,
     10000, 10000, 0, 0, 0, 0, 0, 0, 0, 0},
    {0, 0, 8192, 8192, 8192, 4096, 4096, 4096, 4096, 4096, 4096,
     4096, 4096, 0, 0, 0, 0, 0, 0, 0, 0}};

// The fused form.  Below the limit the staged form's time is the sum of its stages'
// slowest items, which the fused form's slowest whole path undercuts.  It keeps a
// whole mixture on one lane pair, so above nc 12, where the staged form moves the
// trust-region work onto lane groups and the fused form's tail has no teams, it
// pays off only for smaller batches (n nc <= 400,000).  Measured (MI355X, us, staged /
// fused):
//   flash: nc 2 1223 / 1073 at 300,000, 1324 / 1403 at 400,000; nc 4 1200 / 991 at
//   200,000, 1350 / 1372 at 300,000 (own sets 1671 / 1347); nc 5 1418 / 1312 at 150,000,
//   1518 / 1709 at 200,000; nc 8 1448 / 1034 at 80,000, 1917 / 1596 at 150,000, 1703 / 2056
//   at 200,000; nc 9 1644 / 1487 at 100,000, 1746 / 1775 at 130,000; nc 10 1918 / 1897 at
//   100,000, 1923 / 2108 at 110,000; nc 12 2682 / 2398 at 60,000, 2695 / 2676 at 80,000 (own
//   sets 2740 / 2386 at 60,000, 2893 / 3105 at 80,000).
//   Stability analysis, which has no tail of teams: nc 8 735 / 733 at 150,000, 782 / 854
//   at 180,000; nc 9 591 / 564 at 90,000, 598 / 599 at 100,000; nc 10 710 / 662 at 90,000,
//   729 / 736 at 100,000; nc 12 (own sets) 952 / 850 at 70,000.
constexpr int64_t kFusedMaxN[2][21] = {
    {0, 0, 300000, 300000, 300000, 150000, 150000, 150000, 150000, 120000, 100000,
     70000, 70000, 30769, 28571, 26666, 25000, 23529, 22222, 21052, 20000},
    {0, 0, 300000, 300000, 300000, 150000, 150000, 150000, 150000, 90000, 90000,
     70000, 70000, 30769, 28571, 26666, 25000, 23529, 22222, 21052, 20000}};

}  // namespace ptf
