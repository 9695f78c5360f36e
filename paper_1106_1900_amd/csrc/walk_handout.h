// walk_handout.h - the order in which a walk takes the groups, and which of them whole
// workgroups take.  Rules only, for the device and for tests on the host.
//
// A group's time grows with its size, up to several times the mean, so a launch ends with
// wavefronts idle behind the last large groups: all of a small launch, a tenth of one of
// 55,000 groups.  Against that groups are taken by descending size class, and in
// launches of few groups the large ones are walked first, each by a whole workgroup (a
// team, see walk.hip).  The results do not depend on it bit for bit.
#pragma once

#include <cstdint>

namespace bh {

// Size classes 1..6 of the groups.
constexpr int kGroupClasses = 6;
__host__ __device__ constexpr uint8_t group_class(uint32_t size)
{
    return (uint8_t)(1 + (size >= 9) + (size >= 17) + (size >= 33) + (size >= 49) + (size >= 65));
}

// The class of a group in a cluster of n particles.  A small cluster's groups have short
// lists whatever their size, so they come last and no team walks them: 500 clusters of
// 64 particles take 38 us with a wavefront per group, 60 by teams, 100 of 100 42 and 52, 30
// of 300 50 and 52; 10 of 500 57 and 51.
constexpr uint32_t kSmallCluster = 320;
__host__ __device__ constexpr uint8_t group_class(uint32_t size, uint32_t n)
{
    return n <= kSmallCluster ? (uint8_t)1 : group_class(size);
}

// Whether the groups are taken by class (each class in Morton order), of `waves`
// wavefronts in the grid (V; 4096: all that are resident at once).  2^20 particles
// (55,388 groups): 1.69 -> 1.56 ms; 240,002: 0.38 -> 0.29 ms; 81,660 groups 2.50 -> 2.33,
// 80,000 of a galaxy at theta = 0.4 6.64 -> 6.26.  Above, Morton order alone: the groups at
// work then span less of the tree.  Single systems still gain a little by class (119,542
// groups 3.43 and 3.33 ms, 160,000 4.58 and 4.51, 216,204 the same), but the groups of many
// clusters lose more (two steps of 200 clusters of 12,000 particles 4.88 ms in Morton order,
// 5.60 by class, of 400 of 8000 6.32 and 7.35; 470,942 groups 7.97 and 8.6 a walk).
__host__ __device__ constexpr bool by_class(uint64_t ngroups, uint64_t waves)
{
    return ngroups <= 24 * waves;
}

// The smallest class that has its own place in the order; the groups of the classes below
// follow in Morton order together.  With many groups per wavefront the small classes no
// longer shorten the end of a launch, and what neighbours have in common in the tree
// counts, the more the shorter their lists are:
//   up to 8 V    each class by itself: 300,000 particles of a Plummer sphere (4 V, theta =
//                0.4) 2.0 ms in Morton order, 1.57 so, 1.70 with those of up to 32 together;
//                20 clusters of 1000 to 65,536 (6 V) 1.75, 1.47 and 1.57;
//   above        those of up to 16 particles together: 600,000 of a disc galaxy in groups
//                of up to 32 (16 V, theta = 0.75) 0.96, 1.01 and 0.96; 2^20 of a Plummer
//                sphere (13 V) 1.76, 1.64 and 1.65, with up to 32 together 1.68 (at theta =
//                0.4 5.89, 5.30, 5.34 and 5.45);
//   and in clusters of less than 500 groups on average those of up to 48: 300 clusters of
//                1000 to 10,000 (18 V, theta = 0.75) 1.01 in Morton order, 1.15 by all
//                classes, 1.08 with up to 32 and 1.02 with up to 48 together; 60 of 1000
//                to 50,000 (725 groups each, theta = 0.4) 2.35, 2.05, 2.09 and 2.21.
// A single system of many small clumps still loses by it: 1.1M particles in clumps of 200 (17 V)
// 0.87 in Morton order, 0.89 so, by the minimum distance 1.09 and 1.18; 300,000 (4.7 V)
// 0.25 and 0.27.
__host__ __device__ constexpr int first_own_class(uint64_t ngroups, uint64_t waves, uint64_t clusters)
{
    return ngroups <= 8 * waves ? 1 : ngroups < 500 * clusters ? group_class(49) : group_class(17);
}

// Whether groups of 17 to 32 particles have lists too short for a team: by Eq. (1) at a
// large opening angle, in a system without a dense centre (whose tree is shallow).  8192
// particles of a uniform cube, theta = 0.75: 32 us by single wavefronts, 43 by teams from 17
// up; at 0.4, 87 and 68, by the minimum distance 62 and 56.
__host__ __device__ constexpr bool short_lists(uint32_t depth, float theta, uint32_t mac)
{
    return depth < 6 && mac == 0 && theta > 0.55f;
}

// How many groups at the front of the order teams walk; upto[c]: the groups of class c + 1 or
// more.  By the number of groups:
//   up to 4 V     those of 65 and more (two or three particles per lane): 7210 groups of
//                 up to 128: 0.40 -> 0.23 ms;
//   up to 1.5 V   so are those of 49 and more: 5376 groups 0.60 -> 0.54 ms (with 33
//                 and more 0.57: each of a team's wavefronts walks the whole tree);
//   up to 0.625 V so are those of 33 and more: 1891 groups 0.164 -> 0.106 ms;
//   up to 0.25 V  those of 17 and more: 522 groups of up to 64 411 -> 154 us (with 33 and
//                 more 233), 485 of up to 32 133 -> 96.  Not the smaller ones, whose lists
//                 many lanes share already: 4096 particles in groups of up to 16 (1400
//                 of them at most) 91 us so, 79 by teams from 9 up and 151 by teams
//                 from 1 up, 1000 groups of one particle 32 and 93.
// Of these the largest classes that hold no more groups than there are workgroups: where most
// groups are large (a uniform system) they need no help against the tail, and teams walk
// the tree several times for each of them in several rounds.  200,000 particles of a uniform
// cube, 2024 groups of 49 and more of 4572: 143 us so, 202 by teams; 412,977 in groups of up
// to 128, 390 and 465.
__host__ __device__ inline uint32_t team_groups(const uint32_t *upto, uint64_t ngroups, uint64_t waves,
                                                uint32_t workgroups, bool short_lists)
{
    if (ngroups > 4 * waves) return 0;
    int c = group_class(65);
    if (4 * ngroups <= waves) c = group_class(17);
    else if (8 * ngroups <= 5 * waves) c = group_class(33);
    else if (2 * ngroups <= 3 * waves) c = group_class(49);
    if (short_lists && c < group_class(33)) c = group_class(33);
    for (; c <= kGroupClasses; ++c)
        if (upto[c - 1] <= workgroups) return upto[c - 1];
    return 0;
}

}  // namespace bh
