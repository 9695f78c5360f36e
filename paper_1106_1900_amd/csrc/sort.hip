// sort.hip - compaction and the sorts of (key, index) pairs (App. A: count, scan
// offsets, place; stable passes).
//
// Clusters of up to 2^20 particles are sorted through buckets (below): one pass
// that places the pairs by key range and one workgroup per bucket.  A batch with a
// larger cluster, or of thousands of tiny ones (sort_rules.h), takes a stable LSD radix
// sort.  The paper splits one bit per pass;
// here each pass places an 8-bit digit, which is the same stable partition done for
// 256 buckets at once: 8 passes over the 60-bit keys.  For a batch of clusters,
// further stable passes on the cluster of each element follow, so the keys end up
// sorted within each cluster and the clusters keep their places.  Each pass is
// reduce-then-scan (no inter-block waiting):
//   1. hist:    per-block digit counts, stored digit-major;
//   2. scan:    one block per digit scans that digit's counts over blocks;
//   3. scatter: each block ranks its keys stably (wavefront match on the digit
//               bits), stages them in LDS in digit order and writes them out
//               coalesced at digit base + block offset + rank.
#include "bh_internal.h"

#include <algorithm>

namespace bh {
namespace {

// digit of an element: from its key, or (cl != NULL) from the cluster of the
// position it came from
__device__ __forceinline__ uint32_t digit_of(uint64_t k, uint32_t v, const uint32_t *cl, int shift)
{
    return cl ? ((cl[v] >> shift) & (kRadix - 1)) : ((uint32_t)(k >> shift) & (kRadix - 1));
}

// The lanes of the wavefront that are valid and hold the same 8-bit digit as
// this lane: one ballot per digit bit, collecting the lanes that differ.
__device__ __forceinline__ unsigned long long match_digit(uint32_t d, bool valid)
{
    const unsigned long long v = ballot(valid);
    uint32_t dlo = ~(uint32_t)v, dhi = ~(uint32_t)(v >> 32);
#pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
        const uint32_t s = (uint32_t)((int32_t)(d << (31 - b)) >> 31);   // ~0 if bit b is set
        const unsigned long long m = ballot(s != 0u);
        dlo |= (uint32_t)m ^ s;
        dhi |= (uint32_t)(m >> 32) ^ s;
    }
    return ~(((unsigned long long)dhi << 32) | dlo);
}

// OR and AND of a 64-bit value over the wavefront (every lane gets the result)
__device__ __forceinline__ unsigned long long wave_or_u64(unsigned long long v)
{
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) v |= __shfl_xor(v, off);
    return v;
}
__device__ __forceinline__ unsigned long long wave_and_u64(unsigned long long v)
{
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) v &= __shfl_xor(v, off);
    return v;
}

// Exclusive scan of one value per thread over a 256-thread block.  Returns the
// exclusive prefix; *total receives the block sum (same in every thread).
__device__ uint32_t block_excl_scan_256(uint32_t v, uint32_t *s_tmp, uint32_t *total)
{
    const int t = threadIdx.x, w = t / kWave, l = t % kWave;
    uint32_t inc = wave_incl_scan_add(v);
    if (l == kWave - 1) s_tmp[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t x = s_tmp[i];
        if (i < w) off += x;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// The digit of a pass is a radix digit of the key (or of the element's cluster).
__global__ void __launch_bounds__(kSortThreads)
hist_kernel(const uint64_t *__restrict__ keys, const uint32_t *__restrict__ vals,
            const uint32_t *__restrict__ cl, int64_t n, int shift, uint32_t *__restrict__ hist,
            int nblk)
{
    __shared__ uint32_t cnt[kRadix];
    const int t = threadIdx.x;
    cnt[t] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        int64_t i = base + (int64_t)k * kSortThreads + t;
        if (i < n) {
            atomicAdd(&cnt[digit_of(keys[i], cl ? vals[i] : 0u, cl, shift)], 1u);
        }
    }
    __syncthreads();
    hist[(int64_t)t * nblk + blockIdx.x] = cnt[t];
}

// One block per digit: exclusive scan of hist[d][0..nblk) in place, total -> tot[d].
__global__ void __launch_bounds__(256)
scan_digit_kernel(uint32_t *__restrict__ hist, int nblk, uint32_t *__restrict__ tot)
{
    __shared__ uint32_t s_tmp[4];
    uint32_t *row = hist + (int64_t)blockIdx.x * nblk;
    uint32_t run = 0;
    for (int b0 = 0; b0 < nblk; b0 += 256) {
        int b = b0 + threadIdx.x;
        uint32_t v = b < nblk ? row[b] : 0u;
        uint32_t sum;
        uint32_t ex = block_excl_scan_256(v, s_tmp, &sum);
        if (b < nblk) row[b] = run + ex;
        run += sum;
    }
    if (threadIdx.x == 0) tot[blockIdx.x] = run;
}

__global__ void __launch_bounds__(kSortThreads)
scatter_kernel(const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
               uint64_t *__restrict__ kout, uint32_t *__restrict__ vout,
               const uint32_t *__restrict__ cl, int64_t n, int shift,
               const uint32_t *__restrict__ hist, const uint32_t *__restrict__ tot, int nblk)
{
    __shared__ uint32_t s_wcnt[kSortThreads / kWave][kRadix];  // per-wave digit counts
    __shared__ uint32_t s_base[kRadix];                         // global digit base
    __shared__ uint32_t s_local[kRadix];                        // block-local digit start
    __shared__ uint32_t s_tmp[4];
    __shared__ uint64_t s_key[kSortTile];
    __shared__ uint32_t s_val[kSortTile];
    __shared__ uint8_t s_dig[kSortTile];

    const int t = threadIdx.x, w = t / kWave, l = t % kWave;
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
    const int tile_n = (int)((n - base) < kSortTile ? (n - base) : kSortTile);

    for (int d = t; d < kRadix; d += kSortThreads) {
#pragma unroll
        for (int i = 0; i < kSortThreads / kWave; ++i) s_wcnt[i][d] = 0;
    }
    {
        uint32_t sum;
        uint32_t ex = block_excl_scan_256(tot[t], s_tmp, &sum);
        s_base[t] = ex;
    }
    __syncthreads();

    uint64_t key[kSortItems];
    uint32_t val[kSortItems];
    uint32_t rank[kSortItems];
    uint32_t dig[kSortItems];
    const int wbase = w * kWave * kSortItems;  // this wave's contiguous sub-tile
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        int p = wbase + k * kWave + l;
        bool valid = p < tile_n;
        key[k] = valid ? kin[base + p] : 0ull;
        val[k] = valid ? vin[base + p] : 0u;
        uint32_t d = 0;
        if (valid) d = digit_of(key[k], val[k], cl, shift);
        dig[k] = d;
        const unsigned long long peers = match_digit(d, valid);
        uint32_t before = s_wcnt[w][d];
        int r = mask_rank(peers);
        rank[k] = before + (uint32_t)r;
        wave_sync();
        if (valid && r == 0) s_wcnt[w][d] = before + (uint32_t)__popcll(peers);
        wave_sync();
    }
    __syncthreads();

    // wave offsets within the block, block totals, block-local digit starts
    {
        const int d = t;
        uint32_t run = 0;
#pragma unroll
        for (int i = 0; i < kSortThreads / kWave; ++i) {
            uint32_t c = s_wcnt[i][d];
            s_wcnt[i][d] = run;
            run += c;
        }
        uint32_t sum;
        uint32_t ex = block_excl_scan_256(run, s_tmp, &sum);
        s_local[d] = ex;
    }
    __syncthreads();

#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        int p = wbase + k * kWave + l;
        if (p < tile_n) {
            const uint32_t d = dig[k];
            uint32_t lp = s_local[d] + s_wcnt[w][d] + rank[k];
            s_key[lp] = key[k];
            s_val[lp] = val[k];
            s_dig[lp] = (uint8_t)d;
        }
    }
    __syncthreads();

    for (int p = t; p < tile_n; p += kSortThreads) {
        uint64_t k = s_key[p];
        const uint32_t d = s_dig[p];
        int64_t g = (int64_t)s_base[d] + hist[(int64_t)d * nblk + blockIdx.x] + (p - s_local[d]);
        kout[g] = k;
        vout[g] = s_val[p];
    }
}

__global__ void __launch_bounds__(256)
copy_pairs_kernel(const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                  uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) {
        kout[i] = kin[i];
        vout[i] = vin[i];
    }
}

// ---------------------------------------------------------------------------
// generic exclusive scan of u32 / compaction of u8 flags

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;       // flags of a thread: one 64-bit load
constexpr int kScanTile = kScanThreads * kScanItems;
static_assert(kScanTile < 1 << 16, "two counts of a block in one word");

// Counts of the classes 1..kGroupClasses in a block, two 16-bit fields a word
constexpr int kClassWords = (kGroupClasses + 1) / 2;
struct ClassCounts {
    uint32_t w[kClassWords];
};

__device__ __forceinline__ void add_flag(ClassCounts &c, uint8_t f)
{
#pragma unroll
    for (int q = 0; q < kClassWords; ++q)
        c.w[q] += f == 2 * q + 1 ? 1u : (f == 2 * q + 2 ? 1u << 16 : 0u);
}

// a thread's flags of a tile (0 past the end); the tiles begin at multiples of 8
__device__ __forceinline__ void load_flags(const uint8_t *__restrict__ in, int64_t base, int64_t n,
                                           uint8_t *f)
{
    if (base + kScanItems <= n) {
        const uint64_t v = *reinterpret_cast<const uint64_t *>(in + base);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) f[k] = (uint8_t)(v >> (8 * k));
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) f[k] = base + k < n ? in[base + k] : (uint8_t)0;
    }
}

__device__ __forceinline__ uint32_t class_count(const ClassCounts &c, int k)
{
    return (k & 1) ? c.w[k / 2] >> 16 : c.w[k / 2] & 0xffffu;
}

// part[b]: the flags of each class in block b
__global__ void __launch_bounds__(kScanThreads)
scan_reduce_kernel(const uint8_t *__restrict__ in, int64_t n, ClassCounts *__restrict__ part)
{
    __shared__ uint32_t s_tmp[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    ClassCounts c{};
    uint8_t f[kScanItems];
    load_flags(in, base, n, f);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) add_flag(c, f[k]);
    ClassCounts sum;
#pragma unroll
    for (int q = 0; q < kClassWords; ++q) block_excl_scan_256(c.w[q], s_tmp, &sum.w[q]);
    if (threadIdx.x == 0) part[blockIdx.x] = sum;
}

// pre[c nblk + b]: the flags of class c + 1 in the blocks before b; pre[classes nblk + c]: in
// all blocks.  One workgroup per class.
constexpr int kClassScanThreads = 1024;

__global__ void __launch_bounds__(kClassScanThreads)
class_scan_kernel(const ClassCounts *__restrict__ part, uint32_t nblk, uint32_t *__restrict__ pre)
{
    constexpr int kWaves = kClassScanThreads / kWave, kItems = 8;
    __shared__ uint32_t s_tmp[kWaves];
    const int cls = (int)blockIdx.x, t = threadIdx.x, w = t / kWave;
    uint32_t *row = pre + (int64_t)cls * nblk;
    uint32_t run = 0;
    for (uint32_t b0 = 0; b0 < nblk; b0 += kClassScanThreads * kItems) {
        const uint32_t b = b0 + (uint32_t)t * kItems;
        uint32_t v[kItems], mine = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) v[k] = b + k < nblk ? class_count(part[b + k], cls) : 0u;
#pragma unroll
        for (int k = 0; k < kItems; ++k) mine += v[k];
        const uint32_t inc = wave_incl_scan_add(mine);
        if (t % kWave == kWave - 1) s_tmp[w] = inc;
        __syncthreads();
        uint32_t off = 0, sum = 0;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) {
            const uint32_t x = s_tmp[i];
            if (i < w) off += x;
            sum += x;
        }
        __syncthreads();
        uint32_t at = run + off + inc - mine;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            if (b + k < nblk) row[b + k] = at;
            at += v[k];
        }
        run += sum;
    }
    if (t == 0) pre[(int64_t)kGroupClasses * nblk + cls] = run;
}

// Writes the positions of set flags, in order, to idx[0..count), and the same items
// (their positions, or with rank their places in idx) to order: the highest class
// first, each class in order, those below first_own_class as one.  The class counts of
// the blocks before a block and of all blocks come from class_scan_kernel (pre), or, where
// that is null, each block adds up the blocks' counts (part, from scan_reduce_kernel) or,
// where that is null too, counts the flags itself.  The last block also writes count and
// upto[c] = the items of class c + 1 or more.
__global__ void __launch_bounds__(kScanThreads)
compact_down_kernel(const uint8_t *__restrict__ flags, int64_t n,
                    const ClassCounts *__restrict__ part, const uint32_t *__restrict__ pre,
                    uint32_t *__restrict__ idx, uint32_t *__restrict__ count,
                    uint32_t *__restrict__ order, uint32_t *__restrict__ upto, uint32_t waves,
                    uint32_t clusters, bool rank)
{
    __shared__ uint32_t s_tmp[4];
    __shared__ uint32_t s_sum[2][kGroupClasses];    // before this block, in all blocks
    if (threadIdx.x < 2 * kGroupClasses) {
        const uint32_t k = threadIdx.x % kGroupClasses;
        const uint32_t at = threadIdx.x < kGroupClasses ? k * gridDim.x + blockIdx.x
                                                        : kGroupClasses * gridDim.x + k;
        (&s_sum[0][0])[threadIdx.x] = pre ? pre[at] : 0u;
    }
    uint32_t before[kGroupClasses] = {}, all[kGroupClasses] = {};
    if (pre) {
    } else if (part) {
        for (uint32_t b = threadIdx.x; b < gridDim.x; b += kScanThreads) {
            const ClassCounts c = part[b];
#pragma unroll
            for (int k = 0; k < kGroupClasses; ++k) {
                const uint32_t v = class_count(c, k);
                all[k] += v;
                if (b < blockIdx.x) before[k] += v;
            }
        }
    } else {
        for (uint32_t b = 0; b < gridDim.x; ++b) {
            uint8_t f[kScanItems];
            load_flags(flags, (int64_t)b * kScanTile + (int64_t)threadIdx.x * kScanItems, n, f);
            ClassCounts c{};
#pragma unroll
            for (int k = 0; k < kScanItems; ++k) add_flag(c, f[k]);
#pragma unroll
            for (int k = 0; k < kGroupClasses; ++k) {
                const uint32_t v = class_count(c, k);
                all[k] += v;
                if (b < blockIdx.x) before[k] += v;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kGroupClasses; ++k) {
        const uint32_t v = wave_sum_u32(before[k]), t = wave_sum_u32(all[k]);
        if (threadIdx.x % kWave == 0 && t) {
            atomicAdd(&s_sum[0][k], v);
            atomicAdd(&s_sum[1][k], t);
        }
    }
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint8_t f[kScanItems];
    ClassCounts c{}, x;
    uint32_t sum;
    load_flags(flags, base, n, f);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) add_flag(c, f[k]);
#pragma unroll
    for (int q = 0; q < kClassWords; ++q) x.w[q] = block_excl_scan_256(c.w[q], s_tmp, &sum);
    __syncthreads();
    uint32_t run = 0, next[kGroupClasses], first = 0;
    const bool last = blockIdx.x == gridDim.x - 1 && threadIdx.x == 0;
#pragma unroll
    for (int k = kGroupClasses - 1; k >= 0; --k) {
        const uint32_t mine = s_sum[0][k] + class_count(x, k);
        next[k] = first + mine;
        run += mine;
        first += s_sum[1][k];
        if (last) upto[k] = first;
    }
    if (last) *count = first;
    const int own = first_own_class(first, waves, clusters);
    uint32_t back = 0;      // the place of the next item of the classes below it
#pragma unroll
    for (int k = 0; k < kGroupClasses; ++k)
        back += k + 1 < own ? s_sum[0][k] + class_count(x, k) : s_sum[1][k];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (!f[k]) continue;
        const uint32_t item = rank ? run : (uint32_t)(base + k);
        idx[run++] = (uint32_t)(base + k);
#pragma unroll
        for (int q = 0; q < kGroupClasses; ++q)
            if (f[k] == q + 1) order[f[k] < own ? back++ : next[q]++] = item;
    }
}


// ---------------------------------------------------------------------------
// Sort through buckets.  A cluster of one chunk is one bucket.  A larger one gets
// sub buckets per chunk (256 at most), split at keys sampled at about regular places
// of the pairs' order (the candidates, kOver per bucket, written by the keys
// kernel; every place is drawn within its stretch, so that inputs with a period
// of their own are sampled evenly).  One stable pass places the pairs by bucket,
// and one workgroup per bucket sorts it by key, stably.  A load's pairs arrive in
// caller order.  A rebuild's arrive in the held order (the keys kernel writes them
// without the scatter to caller order), and equal keys are then ordered by caller
// index, so the result is the stable sort's of the pairs in caller order, bit for
// bit, either way.
//
// A bucket is a workgroup's LDS sort, so few pairs make little work but the same
// chain of passes: sub is chosen so that the device has a workgroup per CU or two
// (sort_sub).  Loads took eight radix passes (24 launches) before: 100,003
// particles 138 -> 39 us of kernels, 4096 125 -> 23 us.

constexpr uint32_t kOver = kSortOver;   // candidate keys per bucket
static_assert(kRadix == kSortBuckets && kChunk == kSortChunk, "the rule's figures");
constexpr int kWindow = 40;             // bits a bucket's passes cover
constexpr uint32_t kShortRun = 16;      // pairs agreeing in them that one thread orders
constexpr int kPassThreads = 512;       // workgroup of the bucket pass: one chunk
constexpr int kPassItems = kChunk / kPassThreads;
constexpr int kPassWaves = kPassThreads / kWave;
static_assert(kChunk == 4096, "bucket counts below are per 4096 particles");

// The buckets of a cluster, from its record: none of its own pass for one chunk.
__device__ __forceinline__ uint32_t cluster_buckets(const DevCluster &cl, uint32_t sub)
{
    return cl.nchunk > 1 ? cl.nchunk * sub : 1u;
}

// bucket of a key among kRadix - 1 ascending splitters (unused ones are ~0): the
// number of splitters below it, so equal keys share a bucket and buckets follow
// key order; a key that two or more splitters equal has the second one's bucket
// to itself (a bucket of one key needs no sort, however many pairs it holds)
__device__ __forceinline__ uint32_t bucket_of(uint64_t k, const uint64_t *spl)
{
    uint32_t b = 0;
#pragma unroll
    for (uint32_t step = kRadix / 2; step > 0; step >>= 1)
        if (spl[b + step - 1] < k) b += step;
    if (b < kRadix - 2 && spl[b] == k && spl[b + 1] == k) ++b;
    return b;
}

// One workgroup per bucket of a cluster with several chunks: ranks kOver of the
// cluster's candidates against all of them, a wavefront each (ties by index: ranks
// are a permutation); the candidate of rank (b + 1) kOver - 1 becomes splitter b.
// (One workgroup per chunk, with up to 64 candidates: 25 us for 3776 of them, 8 us so.)
__global__ void __launch_bounds__(1024)
splitter_kernel(const Chunk *__restrict__ chunks, const DevCluster *__restrict__ clus, uint32_t sub,
                const uint64_t *__restrict__ cand, uint64_t *__restrict__ spl)
{
    constexpr uint32_t kTile = 2048;
    __shared__ uint64_t s_c[kTile];
    static_assert(kOver == 1024 / kWave, "a wavefront per candidate");
    const uint32_t chunk = blockIdx.x / sub;
    const DevCluster &cl = clus[chunks[chunk].cluster];
    if (cl.nchunk < 2) return;
    const uint32_t nb = cl.nchunk * sub, ncand = nb * kOver;
    const uint64_t *cc = cand + (uint64_t)cl.bucket0 * kOver;
    const uint32_t b = (chunk - cl.chunk0) * sub + blockIdx.x % sub;
    const uint32_t c = b * kOver + threadIdx.x / kWave;
    const uint32_t part = threadIdx.x % kWave;
    const uint64_t mine = cc[c];
    uint32_t below = 0;
    for (uint32_t t0 = 0; t0 < ncand; t0 += kTile) {
        const uint32_t m = min(kTile, ncand - t0);
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < m; i += 1024) s_c[i] = cc[t0 + i];
        __syncthreads();
#pragma unroll 4
        for (uint32_t i = part; i < m; i += kWave) {
            const uint64_t v = s_c[i];
            below += (v < mine || (v == mine && t0 + i < c)) ? 1u : 0u;
        }
    }
    below = wave_sum_u32(below);
    if (part == 0 && (below + 1) % kOver == 0 && (below + 1) / kOver < nb)
        spl[cl.bucket0 + (below + 1) / kOver - 1] = mine;
}

__device__ __forceinline__ void load_splitters(uint64_t *s_spl, const uint64_t *__restrict__ spl,
                                               const DevCluster &cl, uint32_t nb)
{
    for (uint32_t i = threadIdx.x; i < (uint32_t)kRadix; i += blockDim.x)
        s_spl[i] = i + 1 < nb ? spl[cl.bucket0 + i] : ~0ull;
}

// Bucket of every pair (to dig) and the chunk's count of each bucket, stored
// bucket-major per cluster: hist[hist0 + b nchunk + chunk].
__global__ void __launch_bounds__(kPassThreads)
bucket_hist_kernel(const Chunk *__restrict__ chunks, const DevCluster *__restrict__ clus,
                   uint32_t sub, const uint64_t *__restrict__ keys,
                   const uint64_t *__restrict__ spl, uint8_t *__restrict__ dig,
                   uint32_t *__restrict__ hist)
{
    __shared__ uint32_t cnt[kRadix];
    __shared__ uint64_t s_spl[kRadix];
    const Chunk ch = chunks[blockIdx.x];
    const DevCluster &cl = clus[ch.cluster];
    if (cl.nchunk < 2) return;
    const uint32_t nb = cl.nchunk * sub;
    uint64_t key[kPassItems];
#pragma unroll
    for (int k = 0; k < kPassItems; ++k) {
        const uint32_t i = ch.begin + (uint32_t)(k * kPassThreads) + threadIdx.x;
        key[k] = i < ch.end ? keys[i] : 0ull;
    }
    if (threadIdx.x < kRadix) cnt[threadIdx.x] = 0;
    load_splitters(s_spl, spl, cl, nb);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPassItems; ++k) {
        const uint32_t i = ch.begin + (uint32_t)(k * kPassThreads) + threadIdx.x;
        if (i < ch.end) {
            const uint32_t d = bucket_of(key[k], s_spl);
            dig[i] = (uint8_t)d;
            atomicAdd(&cnt[d], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < nb)
        hist[cl.hist0 + threadIdx.x * cl.nchunk + (blockIdx.x - cl.chunk0)] = cnt[threadIdx.x];
}

// One wavefront per bucket: exclusive scan of its counts over the cluster's (at most
// 256) chunks in place, total -> tot.
__global__ void __launch_bounds__(kWave)
bucket_scan_kernel(const Chunk *__restrict__ chunks, const DevCluster *__restrict__ clus,
                   uint32_t sub, uint32_t *__restrict__ hist, uint32_t *__restrict__ tot)
{
    const uint32_t c = blockIdx.x / sub;
    const DevCluster &cl = clus[chunks[c].cluster];
    if (cl.nchunk < 2) return;
    const uint32_t b = (c - cl.chunk0) * sub + blockIdx.x % sub;
    uint32_t *row = hist + cl.hist0 + b * cl.nchunk;
    uint32_t v[4], run = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t i = (uint32_t)(k * kWave) + threadIdx.x;
        v[k] = i < cl.nchunk ? row[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t i = (uint32_t)(k * kWave) + threadIdx.x;
        const uint32_t inc = wave_incl_scan_add(v[k]);
        if (i < cl.nchunk) row[i] = run + inc - v[k];
        run += lane_value(inc, kWave - 1);
    }
    if (threadIdx.x == 0) tot[cl.bucket0 + b] = run;
}

// first position of bucket b of a cluster relative to the cluster (all lanes of the
// calling wavefront; nb buckets of at most kRadix)
__device__ __forceinline__ uint32_t bucket_first(const uint32_t *__restrict__ tot, uint32_t b)
{
    uint32_t x = 0;
    for (uint32_t d = threadIdx.x % kWave; d < b; d += kWave) x += tot[d];
    return wave_sum_u32(x);
}

// The pairs of a chunk to their buckets, stably.
__global__ void __launch_bounds__(kPassThreads)
bucket_scatter_kernel(const Chunk *__restrict__ chunks, const DevCluster *__restrict__ clus,
                      uint32_t sub, const uint64_t *__restrict__ kin,
                      const uint32_t *__restrict__ vin, uint64_t *__restrict__ kout,
                      uint32_t *__restrict__ vout, const uint8_t *__restrict__ dig,
                      const uint32_t *__restrict__ hist, const uint32_t *__restrict__ tot)
{
    __shared__ uint32_t s_wcnt[kPassWaves][kRadix];     // per-wave bucket counts
    __shared__ uint32_t s_out[kRadix];                  // where the chunk's run of a bucket goes
    __shared__ uint32_t s_local[kRadix];                // chunk-local bucket start
    __shared__ uint32_t s_tmp[2][kRadix / kWave];
    __shared__ uint64_t s_key[kChunk];
    __shared__ uint32_t s_val[kChunk];
    __shared__ uint8_t s_dig[kChunk];
    const Chunk ch = chunks[blockIdx.x];
    const DevCluster &cl = clus[ch.cluster];
    if (cl.nchunk < 2) return;
    const uint32_t nb = cl.nchunk * sub;
    const int t = threadIdx.x, w = t / kWave, l = t % kWave;
    const int n = (int)(ch.end - ch.begin);
    uint64_t key[kPassItems];
    uint32_t val[kPassItems], rank[kPassItems], d[kPassItems];
    const int wbase = w * kWave * kPassItems;       // this wave's contiguous part
#pragma unroll
    for (int k = 0; k < kPassItems; ++k) {
        const int p = wbase + k * kWave + l;
        key[k] = p < n ? kin[ch.begin + p] : 0ull;
        val[k] = p < n ? vin[ch.begin + p] : 0u;
        d[k] = p < n ? dig[ch.begin + p] : 0u;
    }
    uint32_t total = 0, before = 0;
    if (t < (int)nb) {
        total = tot[cl.bucket0 + t];
        before = hist[cl.hist0 + (uint32_t)t * cl.nchunk + (blockIdx.x - cl.chunk0)];
    }
    for (int q = t; q < kPassWaves * kRadix; q += kPassThreads) (&s_wcnt[0][0])[q] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPassItems; ++k) {
        const bool valid = wbase + k * kWave + l < n;
        const unsigned long long peers = match_digit(d[k], valid);
        const uint32_t run = s_wcnt[w][d[k]];
        const int r = mask_rank(peers);
        rank[k] = run + (uint32_t)r;
        wave_sync();
        if (valid && r == 0) s_wcnt[w][d[k]] = run + (uint32_t)__popcll(peers);
        wave_sync();
    }
    __syncthreads();
    // wave offsets within the chunk; bucket starts within the chunk and the cluster
    uint32_t mine = 0, inc_m = 0, inc_t = 0;
    if (t < kRadix) {
#pragma unroll
        for (int i = 0; i < kPassWaves; ++i) {
            const uint32_t c = s_wcnt[i][t];
            s_wcnt[i][t] = mine;
            mine += c;
        }
        inc_m = wave_incl_scan_add(mine);
        inc_t = wave_incl_scan_add(total);
        if (l == kWave - 1) {
            s_tmp[0][w] = inc_m;
            s_tmp[1][w] = inc_t;
        }
    }
    __syncthreads();
    if (t < kRadix) {
        uint32_t om = 0, ot = 0;
        for (int i = 0; i < w; ++i) {
            om += s_tmp[0][i];
            ot += s_tmp[1][i];
        }
        s_local[t] = om + inc_m - mine;
        s_out[t] = cl.first + ot + inc_t - total + before;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPassItems; ++k) {
        if (wbase + k * kWave + l < n) {
            const uint32_t lp = s_local[d[k]] + s_wcnt[w][d[k]] + rank[k];
            s_key[lp] = key[k];
            s_val[lp] = val[k];
            s_dig[lp] = (uint8_t)d[k];
        }
    }
    __syncthreads();
    for (int p = t; p < n; p += kPassThreads) {
        const uint32_t b = s_dig[p];
        const uint32_t g = s_out[b] + (uint32_t)p - s_local[b];
        kout[g] = s_key[p];
        vout[g] = s_val[p];
    }
}

// One workgroup per bucket: its pairs are sorted stably by key into (k0, v0).  They lie
// in (k1, v1), or in (k0, v0) for a cluster's only bucket.  With pid == NULL the pairs
// arrive in caller order; otherwise in the held order (value = held position,
// pid[value] = caller index), and equal keys are put in caller order explicitly.  Up
// to kCap pairs are sorted in LDS by stable 8-bit passes (keys and positions move,
// values are gathered at the end), skipping the digits every key of the bucket
// shares, and what those leave open in a second step (see below).  A larger bucket
// (clustered keys that the sample missed, or one key) is sorted by the workgroup
// with the same passes through (k0, v0) and back.
// A pass costs its workgroup about 3 us whatever it holds (a chain of LDS reads, eight
// ballots, counts and four barriers), so the passes cover only kWindow bits: buckets of
// 1024 pairs 31 -> 23 us, of 4096 44 -> 32 us.  Two workgroups share a CU up to 6144
// pairs: LDS and registers are held to that (4000 buckets of 2048 pairs on average
// took 258 us with all passes, 211 us with workgroups of 1024, 187 us with 512).
template <int kCap, int kThreads, int kWavesPerEu>
__global__ void __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(kWavesPerEu)))
bucket_sort_kernel(const Chunk *__restrict__ chunks, const DevCluster *__restrict__ clus, uint32_t sub,
                   uint64_t *__restrict__ k1, uint32_t *__restrict__ v1, uint64_t *__restrict__ k0,
                   uint32_t *__restrict__ v0, const uint32_t *__restrict__ tot,
                   const uint32_t *__restrict__ pid)
{
    constexpr int kBucketThreads = kThreads, kBucketWaves = kThreads / kWave;
    constexpr int kItems = kCap / kThreads;         // most pairs per thread in LDS
    __shared__ uint64_t s_k[kCap];
    __shared__ uint16_t s_x[kCap];
    __shared__ uint16_t s_wcnt[kBucketWaves][kRadix];
    __shared__ uint16_t s_wcnt2[kBucketWaves][kRadix];     // the next LDS pass's counts
    __shared__ uint32_t s_off[kRadix];
    __shared__ uint32_t s_ctot[kRadix];
    __shared__ uint32_t s_tmp[kBucketWaves];
    __shared__ uint32_t s_lo;
    __shared__ unsigned long long s_or, s_and;
    static_assert(kCap < 1 << 16, "positions and counts of a bucket in 16 bits");
    const int t = threadIdx.x, w = t / kWave, lane = t % kWave;
    const uint32_t chunk = blockIdx.x / sub;
    const DevCluster &cl = clus[chunks[chunk].cluster];
    const uint32_t b = (chunk - cl.chunk0) * sub + blockIdx.x % sub;
    if (b >= cluster_buckets(cl, sub)) return;
    const bool only = cl.nchunk < 2;
    if (only) {
        k1 = k0;
        v1 = v0;
    } else if (w == 0) {       // the bucket's first position: the sizes of the buckets before it
        const uint32_t x = bucket_first(tot + cl.bucket0, b);
        if (lane == 0) s_lo = x;
    }
    __syncthreads();
    const int64_t lo = (int64_t)cl.first + (only ? 0u : s_lo);
    const uint32_t L = only ? cl.n : tot[cl.bucket0 + b];
    const uint32_t first = cl.first;        // a cluster's caller indices start there
    if (L == 0) return;

    if (L <= (uint32_t)kCap) {
        const int items = (int)((L + kBucketThreads - 1) / kBucketThreads);
        const uint32_t sub = (uint32_t)items * kWave;      // a wavefront's positions
        uint16_t(*cur)[kRadix] = s_wcnt;       // counts of a pass (zero at its start)
        uint16_t(*nxt)[kRadix] = s_wcnt2;      // cleared during a pass for the next one
        // s_k[i] = v[j] for positions i = j kBucketThreads + t < L, s_x[i] = i, with
        // every load of the thread in flight at once; returns the bits in which
        // the values differ
        auto load = [&](const uint64_t(&v)[kItems]) -> uint64_t {
            __syncthreads();        // earlier readers of s_k, s_x, s_or and s_and are done
            unsigned long long o = 0ull, a = ~0ull;
#pragma unroll
            for (int j = 0; j < kItems; ++j) {
                const uint32_t i = (uint32_t)(j * kBucketThreads + t);
                if (i < L) {
                    s_k[i] = v[j];
                    s_x[i] = (uint16_t)i;
                    o |= v[j];
                    a &= v[j];
                }
            }
            o = wave_or_u64(o);
            a = wave_and_u64(a);
            if (t == 0) {
                s_or = 0ull;
                s_and = ~0ull;
            }
            for (int q = t; q < kBucketWaves * kRadix; q += kBucketThreads) (&cur[0][0])[q] = 0;
            __syncthreads();
            if (lane == 0) {
                atomicOr(&s_or, o);
                atomicAnd(&s_and, a);
            }
            __syncthreads();
            return s_or ^ s_and;
        };
        // stable 8-bit passes over the bits of s_k from bit `from` up in which vary has
        // bits
        auto passes = [&](uint64_t vary, int from) {
            for (int shift = from; shift < 64; shift += kRadixBits) {
                if (((vary >> shift) & (kRadix - 1)) == 0) continue;    // one digit: order kept
                // thread (w, lane) takes positions w sub + j kWave + lane: position
                // order is (wavefront, j, lane) order, which the ranks below keep
                uint64_t key[kItems];
                uint32_t idx[kItems], rank[kItems], dg[kItems];
#pragma unroll
                for (int j = 0; j < kItems; ++j) {
                    if (j < items) {    // uniform
                        const uint32_t p = w * sub + (uint32_t)(j * kWave + lane);
                        const bool valid = p < L;
                        key[j] = valid ? s_k[p] : 0ull;
                        idx[j] = valid ? s_x[p] : 0u;
                        const uint32_t d = (uint32_t)(key[j] >> shift) & (kRadix - 1);
                        dg[j] = d;
                        const unsigned long long peers = match_digit(d, valid);
                        const int r = mask_rank(peers);
                        const uint32_t before = j == 0 ? 0u : cur[w][d];
                        rank[j] = before + (uint32_t)r;
                        wave_sync();
                        if (valid && r == 0) cur[w][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
                        wave_sync();
                    }
                }
                for (int q = t; q < kBucketWaves * kRadix; q += kBucketThreads) (&nxt[0][0])[q] = 0;
                __syncthreads();
                uint32_t cnt = 0, inc = 0;
                if (t < kRadix) {   // wavefronts before each one, per digit; digit totals
                    uint32_t x[kBucketWaves];
#pragma unroll
                    for (int q = 0; q < kBucketWaves; ++q) x[q] = cur[q][t];
                    uint32_t run = 0;
#pragma unroll
                    for (int q = 0; q < kBucketWaves; ++q) {
                        cur[q][t] = (uint16_t)run;
                        run += x[q];
                    }
                    cnt = run;
                    inc = wave_incl_scan_add(cnt);
                    if (lane == kWave - 1) s_tmp[w] = inc;
                }
                __syncthreads();
                if (t < kRadix) {
                    uint32_t before = 0;
                    for (int q = 0; q < w; ++q) before += s_tmp[q];
                    s_off[t] = before + inc - cnt;    // first position of digit t
                }
                __syncthreads();
#pragma unroll
                for (int j = 0; j < kItems; ++j) {
                    const uint32_t p = w * sub + (uint32_t)(j * kWave + lane);
                    if (j < items && p < L) {
                        const uint32_t d = dg[j];
                        const uint32_t np = s_off[d] + cur[w][d] + rank[j];
                        s_k[np] = key[j];
                        s_x[np] = (uint16_t)idx[j];
                    }
                }
                __syncthreads();
                uint16_t(*tmp)[kRadix] = cur;
                cur = nxt;
                nxt = tmp;
            }
        };

        uint64_t v[kItems];
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            const uint32_t i = (uint32_t)(j * kBucketThreads + t);
            v[j] = i < L ? k1[lo + i] : 0ull;
        }
        // The passes cover the kWindow highest bits in which the keys differ.  Pairs that
        // agree in those are still in the order they came in; each short run of them is
        // put in order by the thread of its first pair (by key, and with pid by caller
        // index among equal keys).  A long run has the whole sort done over.
        const uint64_t vary = load(v);
        const int hi = 64 - (int)__clzll((long long)(vary | 1ull));
        const int from = hi > kWindow ? hi - kWindow : 0;
        passes(vary, from);
        bool over = false;
        if (from > 0 || pid) {
            bool tie = false;
            for (uint32_t i = t; i + 1 < L; i += kBucketThreads)
                tie |= (s_k[i] >> from) == (s_k[i + 1] >> from);
            if (__syncthreads_or(tie)) {
                bool lng = false;
                for (uint32_t i = t; i + 1 < L; i += kBucketThreads) {
                    const uint64_t top = s_k[i] >> from;
                    if (top != s_k[i + 1] >> from || (i > 0 && top == s_k[i - 1] >> from)) continue;
                    uint32_t e = i + 2;
                    while (e < L && e - i <= kShortRun && s_k[e] >> from == top) ++e;
                    lng |= e - i > kShortRun;
                }
                over = __syncthreads_or(lng) != 0;
                for (uint32_t i = t; i + 1 < L && !over; i += kBucketThreads) {
                    const uint64_t top = s_k[i] >> from;
                    if (top != s_k[i + 1] >> from || (i > 0 && top == s_k[i - 1] >> from)) continue;
                    // (i's own run: a neighbouring run's pairs differ in the bits above)
                    for (uint32_t e = i + 1; e < L && s_k[e] >> from == top; ++e) {
                        const uint64_t key = s_k[e];
                        const uint16_t x = s_x[e];
                        const uint32_t me = pid ? pid[v1[lo + x]] : 0u;
                        uint32_t q = e;
                        while (q > i && (s_k[q - 1] > key ||
                                         (pid && s_k[q - 1] == key && pid[v1[lo + s_x[q - 1]]] > me))) {
                            s_k[q] = s_k[q - 1];
                            s_x[q] = s_x[q - 1];
                            --q;
                        }
                        s_k[q] = key;
                        s_x[q] = x;
                    }
                }
                __syncthreads();
            }
        }
        if (over) {
            // every bit: without pid from the order now held (pairs of equal keys are
            // still in the order they came in), with it from the caller order
            if (!pid) {
                for (int q = t; q < kBucketWaves * kRadix; q += kBucketThreads) (&cur[0][0])[q] = 0;
                __syncthreads();
                passes(vary, 0);
            } else {
#pragma unroll
                for (int j = 0; j < kItems; ++j) {
                    const uint32_t i = (uint32_t)(j * kBucketThreads + t);
                    v[j] = i < L ? (uint64_t)(pid[v1[lo + i]] - first) : 0ull;
                }
                passes(load(v), 0);     // by caller index
#pragma unroll
                for (int j = 0; j < kItems; ++j) {
                    const uint32_t i = (uint32_t)(j * kBucketThreads + t);
                    v[j] = i < L ? k1[lo + s_x[i]] : 0ull;
                }
                uint16_t x[kItems];
#pragma unroll
                for (int j = 0; j < kItems; ++j) {
                    const uint32_t i = (uint32_t)(j * kBucketThreads + t);
                    x[j] = i < L ? s_x[i] : 0;
                }
                load(v);                            // keys in caller-index order ...
#pragma unroll
                for (int j = 0; j < kItems; ++j) {  // ... with their own positions
                    const uint32_t i = (uint32_t)(j * kBucketThreads + t);
                    if (i < L) s_x[i] = x[j];
                }
                __syncthreads();
                passes(vary, 0);        // then by key
            }
        }
        // every value gather of a thread in flight at once
        uint32_t vout[kItems];
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            const uint32_t i = (uint32_t)(j * kBucketThreads + t);
            // an only bucket's values are its positions as they came
            vout[j] = i < L ? (only ? (uint32_t)lo + s_x[i] : v1[lo + s_x[i]]) : 0u;
        }
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            const uint32_t i = (uint32_t)(j * kBucketThreads + t);
            if (i < L) {
                k0[lo + i] = s_k[i];
                v0[lo + i] = vout[j];
            }
        }
        return;
    }

    // Large bucket (of a cluster with several): stable passes through device memory,
    // (k1, v1) -> (k0, v0) -> (k1, v1) ...: with pid, three passes on the caller index
    // in the cluster (below 2^24) first, then one on each byte in which the keys
    // differ; the result is copied to (k0, v0) if it ends in (k1, v1).
    unsigned long long o = 0ull, a = ~0ull;
    for (uint32_t i = t; i < L; i += kBucketThreads) {
        o |= k1[lo + i];
        a &= k1[lo + i];
    }
    o = wave_or_u64(o);
    a = wave_and_u64(a);
    if (t == 0) {
        s_or = 0ull;
        s_and = ~0ull;
    }
    __syncthreads();
    if (lane == 0) {
        atomicOr(&s_or, o);
        atomicAnd(&s_and, a);
    }
    __syncthreads();
    const uint64_t vary = s_or ^ s_and;
    uint64_t *ks = k1, *kd = k0;
    uint32_t *vs = v1, *vd = v0;
    const int npid = pid ? 3 : 0;
    for (int pass = 0; pass < npid + 8; ++pass) {
        const bool by_pid = pass < npid;
        const int shift = (by_pid ? pass : pass - npid) * kRadixBits;
        if (!by_pid && ((vary >> shift) & (kRadix - 1)) == 0) continue;
        auto digit = [&](uint64_t key, uint32_t val) -> uint32_t {
            return by_pid ? ((pid[val] - first) >> shift) & (kRadix - 1)
                          : (uint32_t)(key >> shift) & (kRadix - 1);
        };
        if (t < kRadix) s_off[t] = 0;
        __syncthreads();
        for (uint32_t i = t; i < L; i += kBucketThreads)
            atomicAdd(&s_off[digit(ks[lo + i], vs[lo + i])], 1u);
        __syncthreads();
        uint32_t cnt = 0, inc = 0;
        if (t < kRadix) {
            cnt = s_off[t];
            inc = wave_incl_scan_add(cnt);
            if (lane == kWave - 1) s_tmp[w] = inc;
        }
        __syncthreads();
        if (t < kRadix) {
            uint32_t before = 0;
            for (int q = 0; q < w; ++q) before += s_tmp[q];
            s_off[t] = before + inc - cnt;        // first output slot of digit t
        }
        __syncthreads();
        for (uint32_t c0 = 0; c0 < L; c0 += kBucketThreads) {
            const uint32_t i = c0 + t;
            const bool valid = i < L;
            const uint64_t key = valid ? ks[lo + i] : 0ull;
            const uint32_t val = valid ? vs[lo + i] : 0u;
            const uint32_t d = valid ? digit(key, val) : 0u;
            const unsigned long long peers = match_digit(d, valid);
            const int r = mask_rank(peers);
            for (int q = t; q < kBucketWaves * kRadix; q += kBucketThreads) (&s_wcnt[0][0])[q] = 0;
            __syncthreads();
            if (valid && r == 0) s_wcnt[w][d] = (uint16_t)__popcll(peers);
            __syncthreads();
            if (t < kRadix) {   // wavefronts before each one, per digit
                uint32_t x[kBucketWaves];
#pragma unroll
                for (int q = 0; q < kBucketWaves; ++q) x[q] = s_wcnt[q][t];
                uint32_t run = 0;
#pragma unroll
                for (int q = 0; q < kBucketWaves; ++q) {
                    s_wcnt[q][t] = (uint16_t)run;
                    run += x[q];
                }
                s_ctot[t] = run;
            }
            __syncthreads();
            if (valid) {
                const uint32_t pos = s_off[d] + s_wcnt[w][d] + (uint32_t)r;
                kd[lo + pos] = key;
                vd[lo + pos] = val;
            }
            __syncthreads();
            if (t < kRadix) s_off[t] += s_ctot[t];
            __syncthreads();
        }
        uint64_t *kt = ks;
        ks = kd;
        kd = kt;
        uint32_t *vt = vs;
        vs = vd;
        vd = vt;
    }
    if (ks != k0) {
        for (uint32_t i = t; i < L; i += kBucketThreads) {
            k0[lo + i] = ks[lo + i];
            v0[lo + i] = vs[lo + i];
        }
    }
}

}  // namespace

namespace {

hipError_t radix_sort_pairs(bh_ctx *c)
{
    const int64_t n = c->n;
    const int nblk = (int)((n + kSortTile - 1) / kSortTile);
    uint32_t *hist = c->blk;                 // kRadix * nblk
    uint32_t *tot = c->blk + (int64_t)kRadix * nblk;
    int cluster_passes = 0;
    for (int64_t k = c->K - 1; k > 0; k >>= kRadixBits) ++cluster_passes;
    const int passes = 8 + cluster_passes;
    int src = 0;
    for (int pass = 0; pass < passes; ++pass) {
        const bool by_cluster = pass >= 8;
        const int shift = by_cluster ? (pass - 8) * kRadixBits : pass * kRadixBits;
        const uint32_t *cl = by_cluster ? c->pcl : nullptr;
        hipLaunchKernelGGL(hist_kernel, dim3(nblk), dim3(kSortThreads), 0, c->stream,
                           c->key[src], c->val[src], cl, n, shift, hist, nblk);
        BH_LAUNCH_CHECK();
        hipLaunchKernelGGL(scan_digit_kernel, dim3(kRadix), dim3(256), 0, c->stream, hist, nblk,
                           tot);
        BH_LAUNCH_CHECK();
        hipLaunchKernelGGL(scatter_kernel, dim3(nblk), dim3(kSortThreads), 0, c->stream,
                           c->key[src], c->val[src], c->key[src ^ 1], c->val[src ^ 1], cl, n, shift,
                           hist, tot, nblk);
        BH_LAUNCH_CHECK();
        src ^= 1;
    }
    if (src != 0) {
        // keep the result in buffer 0 whatever the number of passes
        hipLaunchKernelGGL(copy_pairs_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                           c->stream, c->key[1], c->val[1], c->key[0], c->val[0], n);
        BH_LAUNCH_CHECK();
    }
    return hipSuccess;
}

}  // namespace

int sort_sub(const bh_ctx *c) { return sort_rule(c->n, c->nchunks, c->max_cluster); }

// candidates and splitters, in the cells' centres of mass (written again after the sort)
uint64_t *sort_candidates(bh_ctx *c)
{
    return reinterpret_cast<uint64_t *>(c->c_com) + c->nbuckets;
}

template <int kCap, int kThreads, int kWavesPerEu>
void bucket_sort_launch(bh_ctx *c, uint32_t sub, const uint32_t *tot, const uint32_t *pid)
{
    hipLaunchKernelGGL((bucket_sort_kernel<kCap, kThreads, kWavesPerEu>),
                       dim3((unsigned)(c->nchunks * sub)), dim3(kThreads), 0, c->stream, c->chunks,
                       c->clus, sub, c->key[1], c->val[1], c->key[0], c->val[0], tot, pid);
}

hipError_t sort_pairs(bh_ctx *c, bool held)
{
    const int sub_max = sort_sub(c);
    if (!sub_max) return radix_sort_pairs(c);
    const bool pass = c->nbuckets > 0;
    const uint32_t sub = pass ? (uint32_t)sub_max : 1u;
    uint32_t *hist = c->blk;
    uint32_t *tot = c->blk + c->nhist;
    if (pass) {
        const unsigned g = (unsigned)c->nchunks;
        uint64_t *spl = reinterpret_cast<uint64_t *>(c->c_com);
        hipLaunchKernelGGL(splitter_kernel, dim3(g * sub), dim3(1024), 0, c->stream, c->chunks, c->clus,
                           sub, sort_candidates(c), spl);
        BH_LAUNCH_CHECK();
        hipLaunchKernelGGL(bucket_hist_kernel, dim3(g), dim3(kPassThreads), 0, c->stream, c->chunks,
                           c->clus, sub, c->key[0], spl, c->split, hist);
        BH_LAUNCH_CHECK();
        hipLaunchKernelGGL(bucket_scan_kernel, dim3(g * sub), dim3(kWave), 0, c->stream, c->chunks,
                           c->clus, sub, hist, tot);
        BH_LAUNCH_CHECK();
        hipLaunchKernelGGL(bucket_scatter_kernel, dim3(g), dim3(kPassThreads), 0, c->stream,
                           c->chunks, c->clus, sub, c->key[0], c->val[0], c->key[1], c->val[1],
                           c->split, hist, tot);
        BH_LAUNCH_CHECK();
    }
    // a single chunk is a bucket of up to 4096; others three to four times their mean
    const uint32_t *pid = held ? c->pid[c->cur] : nullptr;
    if (sub_max == 4) bucket_sort_launch<4096, 1024, 8>(c, sub, tot, pid);
    else if (sub_max == 2) bucket_sort_launch<6144, 512, 4>(c, sub, tot, pid);
    else bucket_sort_launch<12288, 1024, 4>(c, sub, tot, pid);
    BH_LAUNCH_CHECK();
    return hipSuccess;
}

// Blocks that count all flags themselves rather than take a launch to count them first
// (4.5 us; each block then reads the others' flags, 8 bytes a thread and block).
constexpr int kCountBlocks = 4;

// Blocks above which their counts are scanned by a launch of their own: otherwise every
// block reads all the others' (12 bytes each), which is quadratic.  Tree and groups of 10^8
// particles 5.92 -> 4.53 ms, of 2^24 837 -> 799 us, of 2^23 420 -> 413; 2^22 the same, and
// below the launch costs 2 us more than it saves.
constexpr int kScanBlocks = 2048;

// the counts of a block of kScanTile flags fit the level rows of its tiles
static_assert((kClassWords + kGroupClasses) * kTreeTile <= (kLevels + 1) * kScanTile &&
              kClassWords + 2 * kGroupClasses <= 2 * (kLevels + 1), "room for the compaction's counts");

hipError_t compact_flags(bh_ctx *c, const uint8_t *flags, int64_t n, uint32_t *idx,
                         uint32_t *count, uint32_t *order, uint32_t *upto, bool rank)
{
    // one block at least, so that the counts are written for n = 0 too
    const int nblk = std::max(1, (int)((n + kScanTile - 1) / kScanTile));
    // in the place of the level rows, which the cells have been made from
    ClassCounts *part = nullptr;
    uint32_t *pre = nullptr;
    if (nblk > kCountBlocks) {
        part = reinterpret_cast<ClassCounts *>(c->blk);
        hipLaunchKernelGGL(scan_reduce_kernel, dim3(nblk), dim3(kScanThreads), 0, c->stream, flags, n,
                           part);
        BH_LAUNCH_CHECK();
    }
    if (nblk > kScanBlocks) {
        pre = reinterpret_cast<uint32_t *>(part + nblk);
        hipLaunchKernelGGL(class_scan_kernel, dim3(kGroupClasses), dim3(kClassScanThreads), 0,
                           c->stream, part, (uint32_t)nblk, pre);
        BH_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(compact_down_kernel, dim3(nblk), dim3(kScanThreads), 0, c->stream, flags, n,
                       part, pre, idx, count, order, upto, (uint32_t)c->walk_spill_waves,
                       (uint32_t)c->K, rank);
    BH_LAUNCH_CHECK();
    return hipSuccess;
}

int64_t sort_blk_words(int64_t n)
{
    const int64_t nblk = (n + kSortTile - 1) / kSortTile;
    return (int64_t)kRadix * nblk + kRadix;
}

}  // namespace bh
