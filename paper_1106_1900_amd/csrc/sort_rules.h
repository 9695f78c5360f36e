// sort_rules.h - which sort the pairs of a load or rebuild take (see sort.hip).  The rule
// only, for the library and for tests on the host.
#pragma once

#include <cstdint>

namespace bh {

constexpr int64_t kSortBuckets = 256;   // most buckets of a cluster
constexpr int64_t kSortChunk = 4096;    // particles per chunk

// Buckets per chunk of the clusters with several chunks, of n particles in all, nchunks
// chunks and max_cluster particles in the largest cluster (0: radix sort).  256 buckets
// per cluster are the limit of the pass, so larger clusters have larger buckets.
//   up to 2^18 particles in all: 1024 pairs a bucket.  A bucket's sort is a chain of
//   passes with little work in each, and 256 workgroups fill the device;
//   clusters of up to 2^19: 2048 pairs, two workgroups to a CU;
//   clusters of up to 2^20: 4096 pairs.
// A cluster of one chunk is a bucket, so thousands of tiny clusters are as many workgroups
// that sort next to nothing (13 ns each): the radix sort, whose time goes with the
// particles, is then the faster.  Two steps of batches in us, buckets and radix sort: of
// 2 particles 721 and 692 (6000 clusters), 3060 and 1830 (32,000); of 64 944 and 960
// (8000), 1370 and 1290 (12,000); of 100 3960 and 3930 (12,000), 5220 and 5110 (16,000);
// of 150 14.6 and 14.7 ms (32,000).
constexpr int sort_rule(int64_t n, int64_t nchunks, int64_t max_cluster)
{
    if (max_cluster > kSortBuckets * kSortChunk) return 0;
    if (160 * nchunks - n > 900000) return 0;
    if (n <= kSortBuckets * kSortChunk / 4) return 4;
    return max_cluster <= kSortBuckets * kSortChunk / 2 ? 2 : 1;
}

}  // namespace bh
