// moment_rules.h - how the moments of the cells are split over workgroups (see build.hip).
// Rules only, for the library and for tests on the host.
//
// A workgroup has the cells of a run of particles and passes their moments from level to
// level through LDS, where there is room for a number of cells; a run of more goes through
// device memory, level by level, at 2 us and more a level.  A system has about 4 cells for
// every leaf size of particles, so runs are the shorter the smaller the leaves.
#pragma once

#include <cstdint>

namespace bh {

constexpr int64_t kRunTile = 256;           // particles per tile; a run begins in a tile
constexpr int64_t kFineRuns = 131072;       // most particles with runs of one tile

// The leaf size to choose by: the least of the clusters', or their mean size if less.
constexpr int run_leaf(int64_t n, int64_t k, int nleaf_min)
{
    const int64_t mean = n / k > 1 ? n / k : 1;
    return mean < nleaf_min ? (int)mean : nleaf_min;
}

// About how many cells n particles have below the roots: 0.25 a particle with leaves of 16,
// 0.43 with 8, 0.7 with 4, 1.5 with 1 (Plummer spheres).
constexpr int64_t about_cells(int64_t n, int leaf)
{
    return leaf > 2 ? 4 * n / leaf : 3 * n / 2;
}

// A run's tiles are 1 << run_tiles_log.  Moments of a build and of a refit in us, in runs
// of four tiles, in the runs chosen, and with a launch per level or two:
//   four for leaves of 14 and more (n = 100,003, leaf 16: 41 and 48; 69 and 90), and where a
//   run has the whole system (n = 300, leaf 4: 16 and 20; 22 and 30);
//   up to 131,072 particles (kSpanUnits runs, so one launch for the nodes across runs)
//   one.  Leaf 8, n = 4096: 50 and 44, 32 and 38; 38 and 53.  Leaf 4, n = 5000: 50 and 63,
//   34 and 41; 43 and 58.  Leaf 1, n = 20,000: 86 and 110, 69 and 85; 76 and 107;
//   beyond, two, from 2^19 particles up where the leaves hold 3 and more.  Leaf 4, 2^20: 149
//   and 248, 154 and 203; 151 and 212.  Leaf 8, 2^22: 278 and 497, 280 and 406; 338 and 464.
constexpr int run_tiles_log(int64_t n, int leaf)
{
    if (leaf >= 14 || (n <= 4 * kRunTile && about_cells(n, leaf) <= 440)) return 2;
    if (n <= kFineRuns) return 0;
    return leaf >= 3 && n <= (int64_t)1 << 19 ? 2 : 1;
}

// Runs of n particles at most, whatever the leaves; grows with n.
constexpr int64_t most_runs(int64_t n)
{
    const int64_t fine = (n < kFineRuns ? n : kFineRuns) / kRunTile, two = n / (2 * kRunTile);
    return (fine > two ? fine : two) + 1;
}

// Whether one workgroup takes the whole system (up to 4096 particles, LDS for 1279 cells): no
// launch for the nodes across runs.  Whole builds: 140 us at 1500 particles and 162 at
// 4000; four workgroups and one across them 150 and 168.
constexpr bool one_workgroup(int64_t n, int64_t k, int leaf)
{
    return n <= 4096 && about_cells(n, leaf) + k <= 1279;
}

// Runs of four tiles have 512 threads and LDS for 511 cells up to these sizes, where a
// launch is a few workgroups per CU and the chain in each counts (a build, a refit); above,
// 256 threads and for 463 (303 in a refit), three workgroups to a CU: refits of 2^22
// particles 361 -> 269 us (with a launch per level 373), 2^24 1241 -> 812 (999), a
// uniform cube 1074 -> 540 (696); builds of 2^24 636 -> 582 (781).
constexpr int64_t kWideRuns = (int64_t)1 << 21, kWideRunsBox = (int64_t)1 << 18;

}  // namespace bh
