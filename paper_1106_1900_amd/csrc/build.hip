// build.hip - tree construction on the device: bounding box, integer map and
// Morton keys (App. B), particle reordering ("moving", Sect. 4.1), the cell array
// (Sect. 2.1), links, groups (Sect. 2.2), float64 multipole moments (Sect. 3.2)
// and the opening radius of Eq. (1) (Sect. 3.3).
//
// Every kernel works on a batch of K independent clusters held back to back in
// the particle arrays (K = 1 for a single system).  Each cluster keeps its own
// domain, keys, tree and groups; the cell array holds the cells of all clusters,
// level-major, and within a level in particle order, so each cluster's cells form
// exactly its own (level, key) ordered array, interleaved by level with the
// others.  Level 0 holds the K roots in cluster order.
//
// The paper forms cells level by level: it masks the keys of particles not yet in
// a leaf, groups equal masked keys by compaction, marks cells of at most N_leaf
// particles as leaves and repeats down to the deepest level, then links parents
// and children with binary searches and atomics.  The same cell array is built
// here with a fixed number of launches, independent of the depth:
//
//   split(i)  = first level at which sorted particles i-1 and i fall in
//               different cells (from the common key prefix; 21 if equal keys;
//               0 at the first particle of a cluster);
//   leaf(i)   = the level of the leaf holding particle i: the first level at
//               which the run of particles sharing i's key prefix is at most
//               N_leaf long, or 20 (found from split() within +-N_leaf of i);
//   particle i starts exactly the cells of the levels split(i) .. leaf(i).
//
// Counting those starts per level and block, one scan per level gives every
// cell its position in the (level, key) order, its parent and first child come
// from the per-level ranks of the same particle, and a cell's end is the first
// start after it at the same or a shallower level.  The result is the paper's
// cell array exactly, in its order.
//
// No kernel here needs a count on the host: cell, group and level counts stay in
// device memory and the kernels that depend on them loop over fixed grids, so a
// whole build can be captured in a HIP graph.
#include <algorithm>

#include "bh_internal.h"

#pragma clang fp contract(off)

namespace bh {

namespace {

constexpr int kBlock = 256;
static_assert(kBlock == kChunkThreads, "per-chunk kernels share box_partial");
constexpr int kFixedGrid = 2048;       // grid of the kernels that read their size on the device

__device__ __forceinline__ uint64_t spread3(uint32_t v)
{
    uint64_t x = v & 0xFFFFFu;
    x = (x | (x << 32)) & 0x001F00000000FFFFull;
    x = (x | (x << 16)) & 0x001F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

__device__ __forceinline__ uint32_t compact3(uint64_t x)
{
    x &= 0x1249249249249249ull;
    x = (x ^ (x >> 2)) & 0x10C30C30C30C30C3ull;
    x = (x ^ (x >> 4)) & 0x100F00F00F00F00Full;
    x = (x ^ (x >> 8)) & 0x001F0000FF0000FFull;
    x = (x ^ (x >> 16)) & 0x001F00000000FFFFull;
    x = (x ^ (x >> 32)) & 0x1FFFFFull;
    return (uint32_t)x;
}

__device__ __forceinline__ uint32_t coord_to_int(double x, double lo, double scale)
{
    double d = x - lo;
    double f = d * scale;
    return f >= (double)kQMax ? kQMax : (uint32_t)f;
}

inline int grid_for(int64_t n, int block) { return (int)((n + block - 1) / block); }

// ---------------------------------------------------------------------------


struct AosSrc {
    const double *p;
    __device__ void get3(int64_t i, double *v) const
    {
        v[0] = p[3 * i];
        v[1] = p[3 * i + 1];
        v[2] = p[3 * i + 2];
    }
};
struct P4Src {
    const double4 *p;
    __device__ void get3(int64_t i, double *v) const
    {
        const double4 q = p[i];
        v[0] = q.x;
        v[1] = q.y;
        v[2] = q.z;
    }
};

// cluster of every particle position, from the chunk table
__global__ void __launch_bounds__(kBlock)
cluster_ids_kernel(const Chunk *__restrict__ chunks, uint32_t *__restrict__ pcl)
{
    const Chunk ch = chunks[blockIdx.x];
    for (uint32_t i = ch.begin + threadIdx.x; i < ch.end; i += kBlock) pcl[i] = ch.cluster;
}

// Per-chunk minima and maxima of each axis: part[6 b + k], k = 0..2 minima, 3..5
// maxima.  A non-finite coordinate sets bit 0 of the misc flags.  (A leapfrog
// step's kick-drift kernel writes the same partials of the drifted positions.)
template <typename Src>
__global__ void __launch_bounds__(kBlock)
bbox_kernel(Src src, const Chunk *__restrict__ chunks, double *__restrict__ part, DevMisc *m)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) reset_build_counts(m);
    const Chunk ch = chunks[blockIdx.x];
    double lo[3] = {INFINITY, INFINITY, INFINITY};
    double hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    bool bad = false;
    for (uint32_t i = ch.begin + threadIdx.x; i < ch.end; i += kBlock) {
        double v[3];
        src.get3(i, v);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            bad |= !isfinite(v[k]);
            lo[k] = fmin(lo[k], v[k]);
            hi[k] = fmax(hi[k], v[k]);
        }
    }
    box_partial(lo, hi, bad, part, m);
}

// The cluster's cube by a workgroup, from its chunks' partials: side = largest extent (1 if
// all extents vanish); scale = 2^20 / side.  In thread 0's return value.
__device__ __forceinline__ DevDomain cluster_domain(const double *__restrict__ part,
                                                    const DevCluster &cl)
{
    const uint32_t b0 = cl.chunk0, b1 = cl.chunk0 + cl.nchunk;
    double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (uint32_t b = b0 + threadIdx.x; b < b1; b += kBlock) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            v[k] = fmin(v[k], part[6 * (int64_t)b + k]);
            v[3 + k] = fmax(v[3 + k], part[6 * (int64_t)b + 3 + k]);
        }
    }
    __shared__ double s_v[6][kBlock / kWave];
    const int w = threadIdx.x / kWave, l = threadIdx.x % kWave;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        double a = v[k];
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) {
            const double o = __shfl_xor(a, d, kWave);
            a = k < 3 ? fmin(a, o) : fmax(a, o);
        }
        if (l == 0) s_v[k][w] = a;
    }
    __syncthreads();
    DevDomain d{};
    if (threadIdx.x != 0) return d;
    double side = 0.0;
    for (int k = 0; k < 3; ++k) {
        d.lo[k] = s_v[k][0];
        d.hi[k] = s_v[3 + k][0];
        for (int i = 1; i < kBlock / kWave; ++i) {
            d.lo[k] = fmin(d.lo[k], s_v[k][i]);
            d.hi[k] = fmax(d.hi[k], s_v[3 + k][i]);
        }
        const double e = d.hi[k] - d.lo[k];
        if (e > side) side = e;
    }
    if (side == 0.0) side = 1.0;
    d.L = side;
    d.scale = 1048576.0 / side;
    return d;
}

// One block per cluster (clusters of so many chunks that the keys kernel does not
// reduce the partials itself).
__global__ void __launch_bounds__(kBlock)
domain_kernel(const double *__restrict__ part, const DevCluster *__restrict__ clus,
              DevDomain *__restrict__ dom)
{
    const DevDomain d = cluster_domain(part, clus[blockIdx.x]);
    if (threadIdx.x == 0) dom[blockIdx.x] = d;
}

// Chunks of a cluster up to which every workgroup of the keys kernel reduces the
// partials (up to four 48-byte records a thread, from the L2) and no launch does so
// before it: keys 6.3 -> 8.7 us at 4096 particles, 13.1 -> 14.8 at 2^20 and no change
// at 2^22, where the launch of their own took 4.4 us and more.
constexpr int64_t kKeysChunks = 4 * kBlock;

// Keys of the particles, written in caller order: the pair of the particle at
// position i goes to slot pid[i] (its caller index; pid == null: the positions
// are the caller order, a first load) with value i.  The stable sort that
// follows then orders equal keys by caller index, on a first load and on every
// rebuild alike (App. A: the split primitive keeps the input order).  With
// held != 0 the pair goes to slot i instead (the bucket sort, which orders equal keys
// by pid itself).  With sub > 0 (buckets per chunk) the clusters of several chunks
// also get their candidate splitters: kSortOver keys per bucket, one from each of
// as many equal stretches of the cluster, its place drawn from a hash of its number.
// With part the cluster's cube is reduced here (and written by its first workgroup).
template <typename Src>
__global__ void __launch_bounds__(kBlock)
keys_kernel(Src src, const Chunk *__restrict__ chunks, const double *__restrict__ part,
            DevDomain *__restrict__ dom,
            const uint32_t *__restrict__ pid, uint32_t n, uint64_t *__restrict__ key,
            uint32_t *__restrict__ val, uint32_t held, const DevCluster *__restrict__ clus,
            uint32_t sub, uint64_t *__restrict__ cand, DevMisc *m)
{
    const Chunk ch = chunks[blockIdx.x];
    __shared__ DevDomain s_dom;
    if (part) {
        const DevCluster &dc = clus[ch.cluster];
        const DevDomain d = cluster_domain(part, dc);
        if (threadIdx.x == 0) {
            s_dom = d;
            if (blockIdx.x == dc.chunk0) dom[ch.cluster] = d;
        }
    } else if (threadIdx.x == 0) {
        s_dom = dom[ch.cluster];
    }
    __syncthreads();
    const DevDomain &cl = s_dom;
    uint32_t ncand = 0, stretch = 1, first = 0;
    if (sub) {
        const DevCluster &dc = clus[ch.cluster];
        if (dc.nchunk > 1) {
            ncand = dc.nchunk * sub * kSortOver;
            stretch = dc.n / ncand;         // 32 or more: a chunk gives 64 candidates at most
            first = dc.first;
            cand += (uint64_t)dc.bucket0 * kSortOver;
        }
    }
    const double inv = 1.0 / (double)stretch;
    const double lx = cl.lo[0], ly = cl.lo[1], lz = cl.lo[2], scale = cl.scale;
    // kKeyBatch elements per thread at a time: all their loads are issued before
    // the scattered stores, which the compiler may not move loads across
    constexpr int kKeyBatch = 8;
    for (uint32_t i0 = ch.begin + threadIdx.x; i0 < ch.end; i0 += kKeyBatch * kBlock) {
        double v[kKeyBatch][3];
        uint32_t o[kKeyBatch];
#pragma unroll
        for (int u = 0; u < kKeyBatch; ++u) {
            const uint32_t i = i0 + (uint32_t)u * kBlock;
            if (i < ch.end) {
                src.get3(i, v[u]);
                o[u] = pid && !held ? pid[i] : i;
            }
        }
#pragma unroll
        for (int u = 0; u < kKeyBatch; ++u) {
            const uint32_t i = i0 + (uint32_t)u * kBlock;
            if (i >= ch.end) continue;
            const uint32_t qx = coord_to_int(v[u][0], lx, scale);
            const uint32_t qy = coord_to_int(v[u][1], ly, scale);
            const uint32_t qz = coord_to_int(v[u][2], lz, scale);
            uint32_t dst = o[u];
            if (dst >= n) {     // caller indices are a permutation of [0, n)
                atomicOr(&m->nonfinite, 8u);
                dst = i;
            }
            const uint64_t k = spread3(qx) | (spread3(qy) << 1) | (spread3(qz) << 2);
            key[dst] = k;
            val[dst] = i;
            if (ncand) {
                const uint32_t j = i - first;
                const uint32_t q = (uint32_t)(((double)j + 0.5) * inv);
                const uint32_t at = (((q * 2654435761u) >> 16) * stretch) >> 16;
                if (q < ncand && j - q * stretch == at) cand[q] = k;
            }
        }
    }
}

__global__ void __launch_bounds__(kBlock)
reorder_from_caller_kernel(const double *__restrict__ pos, const double *__restrict__ mass,
                           const double *__restrict__ vel, const uint32_t *__restrict__ perm,
                           int64_t n, double4 *__restrict__ p4, double4 *__restrict__ v4,
                           uint32_t *__restrict__ pid, DevMisc *m)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int64_t s = perm[i];
    const double ms = mass[s];
    if (!(ms > 0.0) || !isfinite(ms)) atomicOr(&m->nonfinite, 2u);
    p4[i] = make_double4(pos[3 * s], pos[3 * s + 1], pos[3 * s + 2], ms);
    // the velocity record carries the mass too (read by the energy sums)
    v4[i] = vel ? make_double4(vel[3 * s], vel[3 * s + 1], vel[3 * s + 2], ms)
                : make_double4(0.0, 0.0, 0.0, ms);
    pid[i] = (uint32_t)s;
}

__global__ void __launch_bounds__(kBlock)
reorder_kernel(const double4 *__restrict__ p4i, const double4 *__restrict__ v4i,
               const uint32_t *__restrict__ pidi, const uint32_t *__restrict__ perm, int64_t n,
               double4 *__restrict__ p4o, double4 *__restrict__ v4o, uint32_t *__restrict__ pido,
               DevMisc *m)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    uint32_t s = perm[i];
    if (s >= (uint64_t)n) {     // only after an internal error (bit 3 already set)
        atomicOr(&m->nonfinite, 8u);
        s = (uint32_t)i;
    }
    p4o[i] = p4i[s];
    v4o[i] = v4i[s];
    pido[i] = pidi[s];
}

// ---------------------------------------------------------------------------
// cells

__device__ __forceinline__ int wave_min_i32(int v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        const int o = __shfl_xor(v, d, kWave);
        v = o < v ? o : v;
    }
    return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ int wave_max_i32(int v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        const int o = __shfl_xor(v, d, kWave);
        v = o > v ? o : v;
    }
    return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ uint8_t split_level(uint64_t a, uint64_t b)
{
    uint64_t x = a ^ b;
    if (x == 0) return (uint8_t)(kMaxLevel + 1);
    // keys use 60 bits: 4 leading zero bits are not part of the key
    int lz = __clzll((long long)x) - 4;
    return (uint8_t)(1 + lz / 3);
}

// Per particle: split level, leaf level; per block and level: number of cells
// starting in the block.  blk layout: [level][block], then a row of the leaves
// starting in each block.  H is the largest leaf size
// of the batch (the halo); each particle uses its own cluster's leaf size.
__global__ void __launch_bounds__(kTreeTile)
split_leaf_kernel(const uint64_t *__restrict__ key, const uint32_t *__restrict__ pcl, int64_t n,
                  int H, const DevCluster *__restrict__ clus, uint8_t *__restrict__ split,
                  uint8_t *__restrict__ lam, uint8_t *__restrict__ gflag, uint32_t *__restrict__ blk,
                  int nblk, DevMisc *__restrict__ m)
{
    extern __shared__ uint8_t s_dyn[];
    const int W = kTreeTile + 2 * H;              // split values held in LDS
    uint8_t *s_split = s_dyn;                     // [W]
    uint8_t *s_pl = s_dyn + ((W + 15) & ~15);     // [H][kTreeTile] left prefix minima
    __shared__ uint32_t s_cnt[kLevels];
    __shared__ uint32_t s_leaves;

    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kTreeTile;
    if (t < kLevels) s_cnt[t] = 0;
    if (t == 0) s_leaves = 0;
    // split of global index j, with split = 0 at the first particle of a cluster
    // and at n
    for (int u = t; u < W; u += kTreeTile) {
        int64_t j = base - H + u;
        uint8_t v;
        if (j <= 0 || j >= n || pcl[j] != pcl[j - 1]) v = 0;
        else v = split_level(key[j - 1], key[j]);
        s_split[u] = v;
    }
    __syncthreads();

    const int64_t i = base + t;
    const bool valid = i < n;
    uint8_t sp = 0, lm = 0;
    if (valid) {
        const int h = (int)clus[pcl[i]].nleaf;
        sp = s_split[H + t];
        // left prefix minima PL[a] = min split(i - a'), a' = 0..a
        uint8_t run = 255;
        for (int a = 0; a < h; ++a) {
            uint8_t v = (i - a <= 0) ? (uint8_t)0 : s_split[H + t - a];
            run = v < run ? v : run;
            s_pl[a * kTreeTile + t] = run;
        }
        // right prefix minima PR[b] over split(i + b'), b' = 1..b, combined with
        // PL[h - b]: leaf level = min_b max(PL[h - b], PR[b])
        uint8_t best = 255;
        run = 255;
        for (int b = 1; b <= h; ++b) {
            uint8_t v = (i + b >= n) ? (uint8_t)0 : s_split[H + t + b];
            run = v < run ? v : run;
            uint8_t pl = s_pl[(h - b) * kTreeTile + t];
            uint8_t mx = pl > run ? pl : run;
            best = mx < best ? mx : best;
        }
        lm = best > kMaxLevel ? (uint8_t)kMaxLevel : best;
        split[i] = sp;
        lam[i] = lm;
        gflag[i] = 0;       // group starts are flagged later by cell_finish_kernel
    }
    // count starts per level (only the levels where some particle of the
    // wavefront starts a cell)
    const int l = t % kWave;
    const bool starts = valid && sp <= lm;
    const int lo = wave_min_i32(starts ? (int)sp : kLevels);
    const int hi = wave_max_i32(starts ? (int)lm : -1);
    for (int lev = lo; lev <= hi; ++lev) {
        unsigned long long b = ballot(valid && sp <= lev && lev <= lm);
        if (l == 0 && b) atomicAdd(&s_cnt[lev], (uint32_t)__popcll(b));
    }
    {
        unsigned long long b = ballot(valid && sp <= lm);
        if (l == 0 && b) atomicAdd(&s_leaves, (uint32_t)__popcll(b));
    }
    __syncthreads();
    if (t < kLevels) blk[(int64_t)t * nblk + blockIdx.x] = s_cnt[t];
    // leaves started in this block: one more row of the count table, summed by
    // scan_levels_kernel (a device-wide atomic per block serialises at one address)
    if (t == 0) blk[(int64_t)kLevels * nblk + blockIdx.x] = s_leaves;
}

// level counts -> level offsets (level-major order), total cells, depth.
__device__ void level_finalize(const uint32_t *__restrict__ tot, DevMisc *m, int64_t cap_c)
{
    uint64_t off = 0;
    uint32_t depth = 0;
    uint32_t cnt[kLevels];
    for (int l = 0; l < kLevels; ++l) {
        cnt[l] = __hip_atomic_load(&tot[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        m->level_offset[l] = (uint32_t)off;
        m->level_count[l] = cnt[l];
        if (cnt[l]) depth = (uint32_t)l;
        off += cnt[l];
    }
    if (off > (uint64_t)cap_c) {
        // cannot happen for a consistent tree; keep every later write in bounds
        m->nonfinite |= 4u;
        for (int l = 0; l < kLevels; ++l) m->level_count[l] = 0;
        off = 0;
    }
    m->level_offset[kLevels] = (uint32_t)off;
    m->ncells = (uint32_t)off;
    m->depth = depth;
    m->nleaves = __hip_atomic_load(&tot[kLevels], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Up to this many tiles the workgroups of emit_cells_kernel add the rows up themselves, a
// thread per level with all its loads at once, and no launch scans them first: 4096
// particles 7.4 us for scan and cells, 5.9 + 9.5 with two launches.
constexpr int kEmitTiles = 16;

// one block per level (and one for the leaf row): exclusive scan of the row's
// block counts in place; the last block to finish derives the level offsets
constexpr int kScanLevelsBlock = 1024;

__global__ void __launch_bounds__(kScanLevelsBlock)
scan_levels_kernel(uint32_t *__restrict__ blk, int nblk, uint32_t *__restrict__ tot, DevMisc *m,
                   int64_t cap_c)
{
    constexpr int kWaves = kScanLevelsBlock / kWave;
    __shared__ uint32_t s_tmp[kWaves];
    uint32_t *row = blk + (int64_t)blockIdx.x * nblk;
    uint32_t run = 0;
    const int t = threadIdx.x, w = t / kWave, l = t % kWave;
    for (int b0 = 0; b0 < nblk; b0 += kScanLevelsBlock) {
        int b = b0 + t;
        uint32_t v = b < nblk ? row[b] : 0u;
        uint32_t inc = wave_incl_scan_add(v);
        if (l == kWave - 1) s_tmp[w] = inc;
        __syncthreads();
        uint32_t off = 0, totw = 0;
        for (int k = 0; k < kWaves; ++k) {
            const uint32_t x = s_tmp[k];
            if (k < w) off += x;
            totw += x;
        }
        __syncthreads();
        if (b < nblk) row[b] = run + off + inc - v;
        run += totw;
    }
    if (t == 0) {
        __hip_atomic_store(&tot[blockIdx.x], run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // release this level's total, then count the finished levels
        const uint32_t done = __hip_atomic_fetch_add(&m->levels_done, 1u, __ATOMIC_ACQ_REL,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        if (done == gridDim.x - 1) {
            level_finalize(tot, m, cap_c);
            m->levels_done = 0;      // ready for the next build
        }
    }
}

// For every level, the index of the cell of that level holding particle i
// (valid up to lam(i)): level offset + number of starts at that level up to i,
// minus one.  Computed with wavefront ballots and the scanned block counts.
struct Ranks {
    uint32_t anc[kLevels];
};

// Only the levels lo..hi (wavefront-uniform) get their ranks; the starts of every
// level are counted, as other wavefronts of the block may need them.
// base[lev]: the starts of level lev before this block; off[lev]: the level's offset.
__device__ __forceinline__ void level_ranks(bool valid, uint8_t sp, uint8_t lm,
                                            const uint32_t *base, const uint32_t *off0,
                                            uint32_t (*s_wc)[kLevels],
                                            int lo, int hi, Ranks &r)
{
    const int t = threadIdx.x, w = t / kWave, l = t % kWave;
    unsigned long long balls[kLevels];
#pragma unroll
    for (int lev = 0; lev < kLevels; ++lev) {
        balls[lev] = ballot(valid && sp <= lev && lev <= lm);
        if (l == 0) s_wc[w][lev] = (uint32_t)__popcll(balls[lev]);
    }
    __syncthreads();
    const unsigned long long le = (l == kWave - 1) ? ~0ull : ((2ull << l) - 1ull);
#pragma unroll
    for (int lev = 0; lev < kLevels; ++lev) {
        if (lev < lo || lev > hi) continue;
        uint32_t off = base[lev];
        for (int ww = 0; ww < w; ++ww) off += s_wc[ww][lev];
        uint32_t incl = off + (uint32_t)__popcll(balls[lev] & le);
        r.anc[lev] = off0[lev] + incl - 1u;
    }
}

// Where a run of the moments kernels begins: the particle with the lowest split level of
// every first, second or fourth tile (the first of them; see moment_rules.h), so that few
// cells reach across, with that level and the starts of each level before it.
static_assert(kTreeTile == kRunTile, "runs are whole tiles");
struct RunEdge {
    uint32_t x;
    uint32_t split;
    uint32_t c[kLevels];
};

// Every cell a particle starts: its first particle, level, leaf flag, parent and
// first child.  The last particle of a cell (the next particle starts a cell at
// the same or a shallower level, or lies beyond the cluster) writes the cell's
// end; the last particle of a node also writes one past the node's last child
// (the child holding that particle).  Counts follow as end - first.
// kScan: the rows of blk are not scanned yet, and this kernel does it (see kEmitTiles).
template <bool kScan>
__global__ void __launch_bounds__(kTreeTile)
emit_cells_kernel(const uint8_t *__restrict__ split, const uint8_t *__restrict__ lam, int64_t n,
                  const uint32_t *__restrict__ blk, int nblk, DevMisc *__restrict__ m,
                  int64_t cap_c, uint32_t *__restrict__ c_first, uint8_t *__restrict__ c_level,
                  uint8_t *__restrict__ c_leaf, uint32_t *__restrict__ c_parent,
                  uint32_t *__restrict__ c_child, uint32_t *__restrict__ c_end,
                  uint32_t *__restrict__ c_cend, const uint32_t *__restrict__ pcl,
                  uint32_t *__restrict__ c_cl, RunEdge *__restrict__ edges, int run_log)
{
    __shared__ uint32_t s_wc[kTreeTile / kWave][kLevels];
    __shared__ int s_edge[kTreeTile / kWave];
    __shared__ uint32_t s_base[kLevels], s_off[kLevels + 1], s_tot[kLevels + 1];
    const int64_t i = (int64_t)blockIdx.x * kTreeTile + threadIdx.x;
    const bool valid = i < n;
    const uint8_t sp = valid ? split[i] : (uint8_t)255;
    const uint8_t lm = valid ? lam[i] : (uint8_t)0;
    // split of the next particle: 0 past the end (and at a cluster's first particle)
    const uint8_t sn = (valid && i + 1 < n) ? split[i + 1] : (uint8_t)0;
    // the levels whose ranks this particle uses: from the parent of its first
    // start or end up to its leaf (none if it starts and ends nothing)
    const int first_lev = sp < sn ? sp : sn;
    const bool used = valid && first_lev <= lm;
    const int lo = wave_min_i32(used ? (first_lev > 0 ? first_lev - 1 : 0) : kLevels);
    const int hi = wave_max_i32(used ? (int)lm : -1);
    const bool edge = (blockIdx.x & ((1u << run_log) - 1u)) == 0u;      // a run begins in this tile
    if (edge) {
        const int k = wave_min_i32(((int)sp << 8) | (int)threadIdx.x);
        if (threadIdx.x % kWave == 0) s_edge[threadIdx.x / kWave] = k;
    }
    if (kScan) {
        if (threadIdx.x < kLevels + 1) {
            const uint32_t *row = blk + (int64_t)threadIdx.x * nblk;
            uint32_t v[kEmitTiles], before = 0, total = 0;
#pragma unroll
            for (int q = 0; q < kEmitTiles; ++q) v[q] = q < nblk ? row[q] : 0u;
#pragma unroll
            for (int q = 0; q < kEmitTiles; ++q) {
                if (q < (int)blockIdx.x) before += v[q];
                total += v[q];
            }
            s_tot[threadIdx.x] = total;
            if (threadIdx.x < kLevels) s_base[threadIdx.x] = before;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t off = 0, depth = 0;
            for (int l = 0; l < kLevels; ++l) {
                s_off[l] = off;
                if (s_tot[l]) depth = (uint32_t)l;
                off += s_tot[l];
            }
            // cannot happen for a consistent tree; keeps every later write in bounds
            const bool over = (int64_t)off > cap_c;
            s_off[kLevels] = over ? 0u : off;
            if (blockIdx.x == 0) {
                for (int l = 0; l < kLevels; ++l) {
                    m->level_offset[l] = s_off[l];
                    m->level_count[l] = over ? 0u : s_tot[l];
                }
                m->level_offset[kLevels] = m->ncells = s_off[kLevels];
                m->depth = depth;
                m->nleaves = s_tot[kLevels];
                if (over) m->nonfinite |= 4u;
            }
        }
    } else {
        if (threadIdx.x < kLevels) {
            s_base[threadIdx.x] = blk[(int64_t)threadIdx.x * nblk + blockIdx.x];
            s_off[threadIdx.x] = m->level_offset[threadIdx.x];
        }
        if (threadIdx.x == 0) s_off[kLevels] = m->ncells;
    }
    // (the barrier of level_ranks comes before the first use of s_base and s_off)
    Ranks r;
    level_ranks(valid, sp, lm, s_base, s_off, s_wc, lo, hi, r);
    if (edge) {
        int k = s_edge[0];
        for (int w = 1; w < kTreeTile / kWave; ++w) k = min(k, s_edge[w]);
        const int t0 = k & 255, l = threadIdx.x % kWave;
        if ((int)threadIdx.x / kWave == t0 / kWave) {       // its wavefront: a lane per level
            RunEdge &e = edges[blockIdx.x >> run_log];
            const unsigned long long lt = (1ull << (t0 % kWave)) - 1ull;
            uint32_t c = 0;
            for (int lev = 0; lev < kLevels; ++lev) {
                const unsigned long long b = ballot(valid && sp <= lev && lev <= lm);
                if (l == lev) c = (uint32_t)__popcll(b & lt);
            }
            if (l < kLevels) {
                c += s_base[l];
                for (int w = 0; w < t0 / kWave; ++w) c += s_wc[w][l];
                e.c[l] = c;
            }
            if (l == 0) {
                e.x = blockIdx.x * kTreeTile + (uint32_t)t0;
                e.split = (uint32_t)(k >> 8);
            }
        }
    }
    const uint32_t ncells = s_off[kLevels];
    if (!valid || ncells == 0) return;
    const uint32_t cluster = sp <= lm ? pcl[i] : 0u;
#pragma unroll
    for (int lev = 0; lev < kLevels; ++lev) {
        if (lev < lo || lev > hi) continue;      // wavefront-uniform
        if (lev > lm) continue;
        const uint32_t c = r.anc[lev];
        if (c >= ncells) continue;
        if (lev >= sp) {
            c_first[c] = (uint32_t)i;
            c_cl[c] = cluster;
            c_level[c] = (uint8_t)lev;
            c_leaf[c] = (uint8_t)(lev == lm);
            c_parent[c] = lev > 0 ? r.anc[lev > 0 ? lev - 1 : 0] : kNone;
            c_child[c] = lev < lm ? r.anc[lev < kMaxLevel ? lev + 1 : kMaxLevel] : kNone;
        }
        if (lev >= sn) {
            // particle i is the last of its level-lev cell
            c_end[c] = (uint32_t)(i + 1);
            if (lev < lm) {
                const uint32_t last = r.anc[lev < kMaxLevel ? lev + 1 : kMaxLevel];
                c_cend[c] = last + 1u;
            }
        }
    }
}

// Per cell: count = end - first, children = one past the last child - first
// child (0 for a leaf), and the group starts (Sect. 2.2): a cell of at most
// ncrit particles whose parent holds more (or the root) starts a group at its
// first particle; a leaf still larger than ncrit is cut into runs of ncrit
// particles.  A start's flag is the group's size class.  Reads the ends of a
// cell's parent, never its converted fields.
__global__ void __launch_bounds__(kBlock)
cell_finish_kernel(DevMisc *__restrict__ m, const uint32_t *__restrict__ pcl,
                   const DevCluster *__restrict__ clus, const uint32_t *__restrict__ c_first,
                   const uint32_t *__restrict__ c_end, const uint8_t *__restrict__ c_leaf,
                   const uint8_t *__restrict__ c_level, const uint32_t *__restrict__ c_parent,
                   const uint32_t *__restrict__ c_child, uint32_t *__restrict__ c_count,
                   uint32_t *__restrict__ c_nchild, uint8_t *__restrict__ gflag, int64_t n)
{
    const uint32_t ncells = m->ncells;
    for (uint32_t c = blockIdx.x * kBlock + threadIdx.x; c < ncells; c += gridDim.x * kBlock) {
        const uint32_t f = c_first[c];
        uint32_t e = c_end[c];
        const bool leaf = c_leaf[c] != 0;
        const uint32_t nc = leaf ? 0u : c_nchild[c] - c_child[c];
        // never for a consistent tree; keeps every later access in bounds
        if (f >= (uint64_t)n || e <= f || e > (uint64_t)n || (!leaf && (nc < 1u || nc > 8u))) {
            c_count[c] = 0;
            c_nchild[c] = 0;
            atomicOr(&m->nonfinite, 8u);
            continue;
        }
        const uint32_t cnt = e - f;
        c_count[c] = cnt;
        c_nchild[c] = nc;
        const DevCluster &cl = clus[pcl[f]];
        const uint32_t ncrit = cl.ncrit, cn = cl.n;
        bool top = c_level[c] == 0;
        if (!top) {
            const uint32_t p = c_parent[c];
            top = p < ncells && c_end[p] - c_first[p] > ncrit;
        }
        if (cnt <= ncrit && top) gflag[f] = group_class(cnt, cn);
        if (leaf && cnt > ncrit)
            for (uint32_t o = 0; o < cnt; o += ncrit)
                gflag[f + o] = group_class(min(ncrit, cnt - o), cn);
    }
}

// group counts and tight boxes: 16 lanes per group, grid-stride over the groups
// counted on the device
__global__ void __launch_bounds__(kBlock)
group_boxes_kernel(const uint32_t *__restrict__ g_first, const DevMisc *__restrict__ m, int64_t n,
                   const double4 *__restrict__ p4, const uint32_t *__restrict__ pcl,
                   uint32_t *__restrict__ g_count, double4 *__restrict__ g_centre,
                   float4 *__restrict__ g_half)
{
    constexpr int kSeg = 16;                       // lanes per group
    const int64_t ngroups = m->ngroups;
    const int l = threadIdx.x % kSeg;
    for (int64_t g0 = (int64_t)blockIdx.x * (kBlock / kSeg); g0 < ngroups;
         g0 += (int64_t)gridDim.x * (kBlock / kSeg)) {
        const int64_t g = g0 + threadIdx.x / kSeg;
        const bool valid = g < ngroups;
        const uint32_t s = valid ? g_first[g] : 0u;
        const uint32_t e = valid ? ((g + 1 < ngroups) ? g_first[g + 1] : (uint32_t)n) : 0u;
        double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
        for (uint32_t j = s + l; j < e; j += kSeg) {
            const double4 p = p4[j];
            lo[0] = fmin(lo[0], p.x); hi[0] = fmax(hi[0], p.x);
            lo[1] = fmin(lo[1], p.y); hi[1] = fmax(hi[1], p.y);
            lo[2] = fmin(lo[2], p.z); hi[2] = fmax(hi[2], p.z);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
#pragma unroll
            for (int d = kSeg / 2; d > 0; d >>= 1) {
                lo[k] = fmin(lo[k], __shfl_xor(lo[k], d, kWave));
                hi[k] = fmax(hi[k], __shfl_xor(hi[k], d, kWave));
            }
        }
        if (valid && l == 0) {
            g_count[g] = e - s;
            // w: the group's cluster, whose root is the level-0 cell of that index
            g_centre[g] = make_double4(0.5 * (lo[0] + hi[0]), 0.5 * (lo[1] + hi[1]),
                                       0.5 * (lo[2] + hi[2]), (double)pcl[s]);
            g_half[g] = make_float4((float)(0.5 * (hi[0] - lo[0])), (float)(0.5 * (hi[1] - lo[1])),
                                    (float)(0.5 * (hi[2] - lo[2])), 0.0f);
        }
    }
}

// ---------------------------------------------------------------------------
// moments: float64 monopole and second moment, level by level from the deepest
// (Sect. 3.2): a leaf from its particles, a node from its children (one level
// deeper, finished before it), both in array order.

// Where the opening radii and walk records go, and what they are computed from.
struct RecOut {
    const DevCluster *clus;
    const DevDomain *dom;
    const uint8_t *c_level;
    const uint32_t *c_cl;     // cluster of each cell
    const uint64_t *skey;     // sorted keys
    float *rcrit2;
    WalkCell *rec;
    double4 *geo;
};

// Eq. (1): r_crit = l/theta + delta with l = L 2^-level and delta the distance of
// the centre of mass from the cell's geometric centre (a refitted cell whose
// particles left it: its tight box's centre and side); stored as float32 r_crit^2,
// together with the rest of the cell's walk record.  theta, the opening test and
// the domain are those of the cell's cluster k; for the minimum-distance test
// r_crit = l/theta and the cube (centre, half side) goes to geo.  f: the cell's
// first particle (its key gives the key prefix); box: the cell's tight box (lo x,
// y, z, hi x, y, z) after a refit, else null.
__device__ __forceinline__ void cell_record(uint32_t c, uint32_t f, int lev, uint32_t k, bool leaf,
                                            uint32_t link, uint32_t info, const double4 cm,
                                            const float *s3, const double *blo, const double *bhi,
                                            const RecOut &ro)
{
    const DevDomain &cl = ro.dom[k];
    const float theta = ro.clus[k].theta;
    const double l = ldexp(cl.L, -lev);
    const uint64_t pre = ro.skey[f] >> (3 * (kMaxLevel - lev));
    const double gx = cl.lo[0] + ((double)compact3(pre) + 0.5) * l;
    const double gy = cl.lo[1] + ((double)compact3(pre >> 1) + 0.5) * l;
    const double gz = cl.lo[2] + ((double)compact3(pre >> 2) + 0.5) * l;
    // After a refit a cell whose particles all still lie in its key cell keeps
    // this geometry; any other cell takes its box's centre and side
    // max(l, largest extent), so that the cube of the opening tests holds every
    // particle of the cell.  The integer map is monotone, so the particles keep
    // the key cell exactly when the box's two ends do.
    double side = l, cx = gx, cy = gy, cz = gz;
    if (blo) {
        const int sh = kMaxLevel - lev;
        const uint32_t cell[3] = {compact3(pre), compact3(pre >> 1), compact3(pre >> 2)};
        bool inside = true;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            inside = inside && blo[q] >= cl.lo[q] && bhi[q] <= cl.hi[q] &&
                     (coord_to_int(blo[q], cl.lo[q], cl.scale) >> sh) == cell[q] &&
                     (coord_to_int(bhi[q], cl.lo[q], cl.scale) >> sh) == cell[q];
        }
        if (!inside) {
            double ext = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) ext = bhi[q] - blo[q] > ext ? bhi[q] - blo[q] : ext;
            side = ext > l ? ext : l;
            cx = 0.5 * (blo[0] + bhi[0]);
            cy = 0.5 * (blo[1] + bhi[1]);
            cz = 0.5 * (blo[2] + bhi[2]);
        }
    }
    double r;
    if (ro.clus[k].mac) {
        // minimum-distance test: the cube (geometric centre, half side) must lie
        // beyond side / theta of the group's box
        r = side / (double)theta;
        ro.geo[c] = make_double4(cx, cy, cz, 0.5 * side);
    } else {
        const double dx = cm.x - cx, dy = cm.y - cy, dz = cm.z - cz;
        const double delta = sqrt((dx * dx + dy * dy) + dz * dz);
        r = side / (double)theta + delta;
    }
    const float r2 = (float)(r * r);
    ro.rcrit2[c] = r2;
    WalkCell w;
    w.cx = cm.x;
    w.cy = cm.y;
    w.cz = cm.z;
    w.mass = (float)cm.w;
    w.rcrit2 = r2;
    w.link = link;
    w.info = leaf ? (info | 0x80000000u) : info;
#pragma unroll
    for (int q = 0; q < 6; ++q) w.s3[q] = s3[q];
    ro.rec[c] = w;
}

// Moments of leaf c from its particles [s, s + n), in array order, by one thread.  Each
// pass over the members loads a run of kRun of them at once (indices past the end
// repeat the last member and are left out of the sums), so a pass costs one memory
// latency per run instead of one per member; the sums keep the members' order.
constexpr int kRun = 8;

// (m: x, y, z of the centre of mass, mass, second moments, then the box with kBox)
template <bool kBox, class Src>
__device__ __forceinline__ void leaf_moments(uint32_t s, uint32_t n, Src p4, double *m)
{
    double M = 0.0, sx = 0.0, sy = 0.0, sz = 0.0;
    double *S = m + 4;
#pragma unroll
    for (int k = 0; k < 6; ++k) S[k] = 0.0;
    double4 q[kRun];
    // the tight box: min and max are exact, so the order of the members does not
    // matter, nor that the last one may repeat
    double blo[3] = {INFINITY, INFINITY, INFINITY}, bhi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (uint32_t r = 0; r < n; r += kRun) {
#pragma unroll
        for (int k = 0; k < kRun; ++k) q[k] = p4[s + min(r + k, n - 1)];
#pragma unroll
        for (int k = 0; k < kRun; ++k)
            if (r + k < n) M = M + q[k].w;
#pragma unroll
        for (int k = 0; k < kRun; ++k) {
            if (r + k < n) {
                sx = sx + q[k].w * q[k].x;
                sy = sy + q[k].w * q[k].y;
                sz = sz + q[k].w * q[k].z;
            }
        }
        if (kBox) {
#pragma unroll
            for (int k = 0; k < kRun; ++k) {
                blo[0] = fmin(blo[0], q[k].x); bhi[0] = fmax(bhi[0], q[k].x);
                blo[1] = fmin(blo[1], q[k].y); bhi[1] = fmax(bhi[1], q[k].y);
                blo[2] = fmin(blo[2], q[k].z); bhi[2] = fmax(bhi[2], q[k].z);
            }
        }
    }
    const double cx = sx / M, cy = sy / M, cz = sz / M;
    for (uint32_t r = 0; r < n; r += kRun) {
        if (n > (uint32_t)kRun) {       // else they are held from the first pass
#pragma unroll
            for (int k = 0; k < kRun; ++k) q[k] = p4[s + min(r + k, n - 1)];
        }
#pragma unroll
        for (int k = 0; k < kRun; ++k) {
            if (r + k < n) {
                const double dx = q[k].x - cx, dy = q[k].y - cy, dz = q[k].z - cz;
                const double w = q[k].w;
                S[0] += w * dx * dx; S[1] += w * dy * dy; S[2] += w * dz * dz;
                S[3] += w * dx * dy; S[4] += w * dx * dz; S[5] += w * dy * dz;
            }
        }
    }
    m[0] = cx;
    m[1] = cy;
    m[2] = cz;
    m[3] = M;
    if (kBox) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            m[10 + k] = blo[k];
            m[13 + k] = bhi[k];
        }
    }
}

template <bool kBox>
__device__ __forceinline__ void leaf_store(uint32_t c, const double *m, double4 *__restrict__ c_com,
                                           double *__restrict__ c_S, double *__restrict__ box)
{
    c_com[c] = make_double4(m[0], m[1], m[2], m[3]);
    double2 *out = reinterpret_cast<double2 *>(c_S + 6 * (int64_t)c);
#pragma unroll
    for (int k = 0; k < 3; ++k) out[k] = make_double2(m[4 + 2 * k], m[5 + 2 * k]);
    if (kBox) {
        double2 *b = reinterpret_cast<double2 *>(box + 6 * (int64_t)c);
#pragma unroll
        for (int k = 0; k < 3; ++k) b[k] = make_double2(m[10 + 2 * k], m[11 + 2 * k]);
    }
}

// Moments of node c from its n <= 8 children [s, s + n) (one level deeper, already done)
// by eight lanes of a wavefront (a team), in array order.  Each lane loads a child and
// forms its terms; lane q of the team then adds the children's terms of sum q one
// after the other, so every sum keeps the children's order.  (A thread per node
// gathers its children's records itself, 64 lanes and as many cache lines to an
// instruction, 40 instructions a node, and does every sum in turn: a level of nodes
// took 5 to 9 us in one workgroup.)
// Every lane of the wavefront calls with its team's node; n = 0: none.
constexpr int kTeam = 8;
constexpr int kTermRow = kWave + 1;     // odd: lanes of a team read different banks
struct TeamTerms {
    double v[6][kTermRow];
};

// the team's sums in lanes q < kQ: the terms of m members added in order
template <int kQ>
__device__ __forceinline__ double team_sum(const TeamTerms &L, int lane, int m)
{
    const int q = lane % kTeam, base = lane - q;
    double v[kTeam], acc = 0.0;
#pragma unroll
    for (int k = 0; k < kTeam; ++k) v[k] = L.v[q < kQ ? q : 0][base + k];
#pragma unroll
    for (int k = 0; k < kTeam; ++k) acc = k < m ? acc + v[k] : acc;
    return acc;
}

// p, Sk, blo, bhi: the lane's child (zeros and an empty box if it has none).  Returns in
// lane q of the team: M, then x, y, z of the centre of mass (q < 4); second moment q;
// bound q of the box (lo x, y, z, hi x, y, z).
struct NodeOut {
    double com, S, box;
};

template <bool kBox>
__device__ __forceinline__ NodeOut node_moments(TeamTerms &L, uint32_t n, const double4 p,
                                                const double *Sk, double *blo, double *bhi)
{
    const int lane = lane_id();
    const int j = lane % kTeam, base = lane - j;
    NodeOut out;
    L.v[0][lane] = p.w;
    L.v[1][lane] = p.w * p.x;
    L.v[2][lane] = p.w * p.y;
    L.v[3][lane] = p.w * p.z;
    wave_sync();
    const double sum = team_sum<4>(L, lane, (int)n);    // M; sums of m x, m y, m z
    wave_sync();
    const double M = __shfl(sum, base, kWave);
    const double com = sum / M;
    const double dx = p.x - __shfl(com, base + 1, kWave), dy = p.y - __shfl(com, base + 2, kWave),
                 dz = p.z - __shfl(com, base + 3, kWave), w = p.w;
    L.v[0][lane] = Sk[0] + w * dx * dx;
    L.v[1][lane] = Sk[1] + w * dy * dy;
    L.v[2][lane] = Sk[2] + w * dz * dz;
    L.v[3][lane] = Sk[3] + w * dx * dy;
    L.v[4][lane] = Sk[4] + w * dx * dz;
    L.v[5][lane] = Sk[5] + w * dy * dz;
    wave_sync();
    out.S = team_sum<6>(L, lane, (int)n);       // xx, yy, zz, xy, xz, yz
    wave_sync();
    out.com = j == 0 ? M : com;
    out.box = 0.0;
    if (kBox) {
        // the union of the children's boxes
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int d = kTeam / 2; d > 0; d >>= 1) {
                blo[i] = fmin(blo[i], __shfl_xor(blo[i], d, kWave));
                bhi[i] = fmax(bhi[i], __shfl_xor(bhi[i], d, kWave));
            }
            if (j == i) out.box = blo[i];
            if (j == i + 3) out.box = bhi[i];
        }
    }
    return out;
}

template <bool kBox>
__device__ __forceinline__ void node_store(const NodeOut &o, uint32_t c, double4 *__restrict__ c_com,
                                           double *__restrict__ c_S, double *__restrict__ box)
{
    const int j = lane_id() % kTeam;
    if (j < 4) reinterpret_cast<double *>(c_com + c)[j == 0 ? 3 : j - 1] = o.com;
    if (j < 6) c_S[6 * (int64_t)c + j] = o.S;
    if (kBox && j < 6) box[6 * (int64_t)c + j] = o.box;
}

// The same for a node whose children [s, s + n) have their moments in device memory.
template <bool kBox>
__device__ __forceinline__ void node_from_memory(TeamTerms &L, uint32_t c, uint32_t s, uint32_t n,
                                                 double4 *__restrict__ c_com,
                                                 double *__restrict__ c_S, double *__restrict__ box)
{
    const uint32_t j = (uint32_t)(lane_id() % kTeam);
    double4 p = make_double4(0.0, 0.0, 0.0, 0.0);
    double Sk[6] = {0, 0, 0, 0, 0, 0};
    double blo[3] = {INFINITY, INFINITY, INFINITY}, bhi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (j < n) {
        p = c_com[s + j];
        const double2 *q = reinterpret_cast<const double2 *>(c_S + 6 * (int64_t)(s + j));
        const double2 a = q[0], b = q[1], d = q[2];
        Sk[0] = a.x; Sk[1] = a.y; Sk[2] = b.x; Sk[3] = b.y; Sk[4] = d.x; Sk[5] = d.y;
        if (kBox) {
            const double2 *bx = reinterpret_cast<const double2 *>(box + 6 * (int64_t)(s + j));
            const double2 b0 = bx[0], b1 = bx[1], b2 = bx[2];
            blo[0] = b0.x; blo[1] = b0.y; blo[2] = b1.x;
            bhi[0] = b1.y; bhi[1] = b2.x; bhi[2] = b2.y;
        }
    }
    const NodeOut o = node_moments<kBox>(L, n, p, Sk, blo, bhi);
    if (n) node_store<kBox>(o, c, c_com, c_S, box);
}

template <bool kBox>
__device__ __forceinline__ void load_moments(uint32_t c, const double4 *__restrict__ c_com,
                                             const double *__restrict__ c_S,
                                             const double *__restrict__ box, double *m)
{
    const double4 cm = c_com[c];
    m[0] = cm.x;
    m[1] = cm.y;
    m[2] = cm.z;
    m[3] = cm.w;
    const double2 *s = reinterpret_cast<const double2 *>(c_S + 6 * (int64_t)c);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double2 v = s[k];
        m[4 + 2 * k] = v.x;
        m[5 + 2 * k] = v.y;
    }
    if (kBox) {
        const double2 *b = reinterpret_cast<const double2 *>(box + 6 * (int64_t)c);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double2 v = b[k];
            m[10 + 2 * k] = v.x;
            m[11 + 2 * k] = v.y;
        }
    }
}

// The opening radius and walk record of cell c (of level lev in cluster k, first
// particle f) from its moments m (see leaf_moments); link, info: see WalkCell.
template <bool kBox>
__device__ __forceinline__ void moments_record(uint32_t c, uint32_t f, int lev, uint32_t k, bool leaf,
                                               uint32_t link, uint32_t info, const double *m,
                                               const RecOut &ro)
{
    float s3[6];            // 3 S in float32
#pragma unroll
    for (int i = 0; i < 6; ++i) s3[i] = (float)(3.0 * m[4 + i]);
    cell_record(c, f, lev, k, leaf, link, info, make_double4(m[0], m[1], m[2], m[3]), s3,
                kBox ? m + 10 : nullptr, kBox ? m + 13 : nullptr, ro);
}

// What the moments kernels read of the cells.
struct CellIn {
    const DevMisc *m;
    const RunEdge *edges;
    uint32_t nedges;            // runs
    int64_t n;
    const uint8_t *lam;         // see split_leaf_kernel
    const uint8_t *leaf;
    const uint32_t *first, *count, *child, *nchild;
    const double4 *p4;
};

// the starts of level lev before run e (all of the level's after the last run)
__device__ __forceinline__ uint32_t starts_before(const CellIn &in, int lev, uint32_t e)
{
    return e < in.nedges ? in.edges[e].c[lev] : in.m->level_count[lev];
}

__device__ __forceinline__ int64_t run_begin(const CellIn &in, uint32_t e)
{
    return e < in.nedges ? (int64_t)in.edges[e].x : in.n;
}

// A barrier that orders LDS only: loads ahead and stores of results stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Moments, opening radii and walk records of every leaf and of every node that lies
// within one workgroup's kRuns runs.  The cells of a level that start in them are
// consecutive, and the runs' edges say which; only the last of them can reach beyond
// (span_moments_kernel does those).  Leaves of all levels first, a
// thread each, then the nodes level by level from the deepest, a team each: a node's
// children lie in the run if the node does.  The moments pass from level to level
// through LDS (stores to device memory and the loads behind them cost a level 2 us),
// a run of more than kCap cells through device memory.  The records, which no other
// cell waits for, come last.  kBox: also the cells' tight boxes (refits).
// Wavefronts per SIMD that the registers leave room for: as many as the LDS does.
constexpr int run_waves(bool box, int threads, int cap)
{
    if (box) return threads == 512 || cap > 303 ? 2 : (cap > 191 ? 3 : 4);
    return threads == 256 ? 3 : 4;
}

template <bool kBox, int kThreads, int kCap, int kRuns, int kTiles>
__global__ void __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(run_waves(kBox, kThreads, kCap))))
run_moments_kernel(CellIn in, double4 *__restrict__ c_com, double *__restrict__ c_S,
                   double *__restrict__ box, RecOut ro)
{
    constexpr uint32_t kTeams = kThreads / kTeam;
    constexpr int kFields = kBox ? 16 : 10;
    static_assert(kCap % 2 == 1, "a cell's fields in different banks");
    // the staged particles (a run's, of kTiles tiles, and as many more as an ordinary leaf
    // can take it past its end), then the moments of the run's cells (see leaf_moments)
    constexpr int kStage = (kRuns == 1 ? kTiles + 1 : kRuns * kTiles) * kTreeTile + 64;
    constexpr int kStore = kFields * kCap + (kThreads / kWave) * 6 * kTermRow;
    __shared__ double4 s_raw[(kStore / 4 + 1) > kStage ? kStore / 4 + 1 : kStage];
    double(*s_m)[kCap] = reinterpret_cast<double(*)[kCap]>(s_raw);
    TeamTerms *s_terms = reinterpret_cast<TeamTerms *>(&s_m[kFields][0]);
    __shared__ uint16_t s_list[kCap];           // the run's leaves (places in the run)
    __shared__ uint32_t s_leaves;
    __shared__ uint16_t s_ch[kCap];             // first child (place in the run)
    __shared__ uint8_t s_nc[kCap];              // children; 0: not a node of the run
    __shared__ uint32_t s_b[kLevels], s_pre[kLevels + 1];
    if (in.m->ncells == 0) return;      // only after an internal error
    const uint32_t e0 = blockIdx.x * kRuns, e1 = e0 + kRuns;
    const int64_t end = run_begin(in, e1);
    const int t = threadIdx.x;
    TeamTerms &L = s_terms[t / kWave];
    if (t < kWave) {
        uint32_t b = 0, e = 0;
        if (t < kLevels) {
            const uint32_t off = in.m->level_offset[t];
            b = off + starts_before(in, t, e0);
            e = off + starts_before(in, t, e1);
            s_b[t] = b;
        }
        const uint32_t inc = wave_incl_scan_add(e - b);
        if (t < kLevels) s_pre[t + 1] = inc;
        if (t == 0) s_pre[0] = 0;
    }
    __syncthreads();
    const uint32_t total = s_pre[kLevels];
    const bool lds = total <= (uint32_t)kCap;
    auto cell_of = [&](uint32_t i, int &lev) -> uint32_t {
        lev = 0;
        while (i >= s_pre[lev + 1]) ++lev;
        return s_b[lev] + (i - s_pre[lev]);
    };
    // a node of the run: all of its particles lie in it
    auto inside = [&](uint32_t i, int lev, uint32_t f, uint32_t cnt) {
        return i + 1 < s_pre[lev + 1] || (int64_t)f + cnt <= end;
    };
    const uint32_t start = (uint32_t)run_begin(in, e0);
    if (lds) {
        const uint32_t staged = (uint32_t)min((int64_t)kStage, in.n - start);
        for (uint32_t i = t; i < staged; i += kThreads) s_raw[i] = in.p4[start + i];
        if (t == 0) s_leaves = 0;
        __syncthreads();
        for (uint32_t i = t; i < total; i += kThreads) {
            int lev;
            const uint32_t c = cell_of(i, lev);
            const bool leaf = in.leaf[c] != 0;
            const uint32_t f = in.first[c], cnt = in.count[c], ch = in.child[c], nc = in.nchild[c];
            s_nc[i] = !leaf && inside(i, lev, f, cnt) ? (uint8_t)min(nc, 8u) : (uint8_t)0;
            if (!leaf) s_ch[i] = (uint16_t)(s_pre[lev + 1] + (ch - s_b[lev + 1]));
            if (leaf && cnt) s_list[atomicAdd(&s_leaves, 1u)] = (uint16_t)i;
        }
        __syncthreads();
        // the moments take the particles' place when the leaves (all of them but in
        // odd trees: the first kThreads) have read them
        const uint32_t leaves = s_leaves;
        double m[kFields];
        if ((uint32_t)t < leaves) {
            int lev;
            const uint32_t c = cell_of(s_list[t], lev);
            const uint32_t f = in.first[c], cnt = in.count[c];
            if (f - start + cnt <= staged) leaf_moments<kBox>(f - start, cnt, s_raw, m);
            else leaf_moments<kBox>(f, cnt, in.p4, m);
            leaf_store<kBox>(c, m, c_com, c_S, box);
        }
        lds_barrier();
        for (uint32_t q = t; q < leaves; q += kThreads) {
            const uint32_t i = s_list[q];
            if (q != (uint32_t)t) {
                int lev;
                const uint32_t c = cell_of(i, lev);
                leaf_moments<kBox>(in.first[c], in.count[c], in.p4, m);
                leaf_store<kBox>(c, m, c_com, c_S, box);
            }
#pragma unroll
            for (int d = 0; d < kFields; ++d) s_m[d][i] = m[d];
        }
    } else {
        for (uint32_t i = t; i < total; i += kThreads) {
            int lev;
            const uint32_t c = cell_of(i, lev);
            const uint32_t f = in.first[c], cnt = in.count[c];
            if (!in.leaf[c] || cnt == 0u) continue;
            double m[kFields];
            leaf_moments<kBox>(f, cnt, in.p4, m);
            leaf_store<kBox>(c, m, c_com, c_S, box);
        }
    }
    // (a wavefront's trips are uniform: its teams past the end have no node)
    const uint32_t team = (uint32_t)t / kTeam, team0 = (uint32_t)t / kWave * (kWave / kTeam);
    const uint32_t j = (uint32_t)t % kTeam;
    int lev = kMaxLevel - 1;            // level 20 holds only leaves
    while (lev >= 0 && s_pre[lev] == s_pre[lev + 1]) --lev;
    if (lds) {
        for (; lev >= 0; --lev) {
            lds_barrier();
            const uint32_t e = s_pre[lev + 1];
            for (uint32_t i0 = s_pre[lev]; i0 + team0 < e; i0 += kTeams) {
                const uint32_t i = i0 + team;
                const uint32_t n = i < e ? s_nc[i] : 0u;
                if (ballot(n != 0u) == 0ull) continue;
                double4 p = make_double4(0.0, 0.0, 0.0, 0.0);
                double Sk[6] = {0, 0, 0, 0, 0, 0};
                double blo[3] = {INFINITY, INFINITY, INFINITY};
                double bhi[3] = {-INFINITY, -INFINITY, -INFINITY};
                if (j < n) {
                    const uint32_t k = s_ch[i] + j;
                    p = make_double4(s_m[0][k], s_m[1][k], s_m[2][k], s_m[3][k]);
#pragma unroll
                    for (int q = 0; q < 6; ++q) Sk[q] = s_m[4 + q][k];
                    if (kBox) {
#pragma unroll
                        for (int q = 0; q < 3; ++q) {
                            blo[q] = s_m[kFields - 6 + q][k];
                            bhi[q] = s_m[kFields - 3 + q][k];
                        }
                    }
                }
                const NodeOut o = node_moments<kBox>(L, n, p, Sk, blo, bhi);
                if (n) {
                    if (j < 4u) s_m[j == 0u ? 3u : j - 1u][i] = o.com;
                    if (j < 6u) s_m[4u + j][i] = o.S;
                    if (kBox && j < 6u) s_m[kFields - 6u + j][i] = o.box;
                    node_store<kBox>(o, s_b[lev] + (i - s_pre[lev]), c_com, c_S, box);
                }
            }
        }
    } else {
        for (; lev >= 0; --lev) {
            __syncthreads();
            const uint32_t e = s_pre[lev + 1];
            for (uint32_t i0 = s_pre[lev]; i0 + team0 < e; i0 += kTeams) {
                const uint32_t i = i0 + team;
                uint32_t n = 0, ch = 0;
                const uint32_t c = s_b[lev] + (i - s_pre[lev]);
                if (i < e && !in.leaf[c] && inside(i, lev, in.first[c], in.count[c])) {
                    ch = in.child[c];
                    n = min(in.nchild[c], 8u);
                }
                node_from_memory<kBox>(L, c, ch, n, c_com, c_S, box);
            }
        }
    }
    if (lds) lds_barrier();
    else __syncthreads();
    for (uint32_t i = t; i < total; i += kThreads) {
        const uint32_t c = cell_of(i, lev);
        const bool leaf = in.leaf[c] != 0;
        const uint32_t f = in.first[c], cnt = in.count[c], kc = ro.c_cl[c];
        const uint32_t ch = in.child[c], nc = in.nchild[c];
        if (cnt == 0u || (!leaf && !inside(i, lev, f, cnt))) continue;
        double m[kFields];
        if (lds) {
#pragma unroll
            for (int k = 0; k < kFields; ++k) m[k] = s_m[k][i];
        } else {
            load_moments<kBox>(c, c_com, c_S, box, m);
        }
        moments_record<kBox>(c, f, lev, kc, leaf, leaf ? f : ch, leaf ? cnt : nc, m, ro);
    }
}

// Units of several sizes: runs (depth 0), about 64 runs (depth 1), about 64 of those
// (depth 2) and so on.  A unit begins at that one of the first 16 lesser units of its 64
// whose edge has the lowest split level, again so that few cells reach across.
constexpr uint32_t kUnitLog = 6, kWindowLog = 4;
constexpr uint32_t kUnitMost = (1u << kUnitLog) + (1u << kWindowLog) - 1;   // lesser units in one

// the first run of unit u
__device__ __forceinline__ uint32_t unit_begin(const CellIn &in, uint32_t depth, uint32_t u)
{
    const uint64_t b = (uint64_t)u << (kUnitLog * depth);
    if (b >= in.nedges) return in.nedges;
    uint32_t best = (uint32_t)b, low = 255;
    // the candidates in order: digits of kWindowLog bits in places of kUnitLog bits
    for (uint32_t k = 0; k < 1u << (kWindowLog * depth); ++k) {
        uint64_t e = b;
        for (uint32_t d = 0; d < depth; ++d)
            e += (uint64_t)((k >> (kWindowLog * d)) & ((1u << kWindowLog) - 1)) << (kUnitLog * d);
        const uint32_t s = e < in.nedges ? in.edges[e].split : 255u;
        if (s < low) {
            low = s;
            best = (uint32_t)e;
        }
    }
    return best;
}

// The nodes that reach beyond a unit but lie within the workgroup's next larger unit
// (kAll: one workgroup, all of the rest): in each level at most one per unit, the last
// cell that starts in it.  Level by level like a run's own nodes; which nodes there are,
// and their children, is looked up for all levels first, for the chain of levels is
// what bounds it.  As units begin between large cells, each launch has a part of the
// tree's levels.
template <bool kBox, int kUnits, int kThreads, bool kAll>
__global__ void __launch_bounds__(kThreads)
span_moments_kernel(CellIn in, uint32_t depth, double4 *__restrict__ c_com, double *__restrict__ c_S,
                    double *__restrict__ box, RecOut ro)
{
    constexpr uint32_t kTeams = kThreads / kTeam;
    static_assert(kUnits <= kThreads && (kAll || kUnits >= (int)kUnitMost), "a thread per unit");
    __shared__ TeamTerms s_terms[kThreads / kWave];
    __shared__ uint32_t s_cell[kMaxLevel][kUnits], s_ch[kMaxLevel][kUnits];
    __shared__ uint8_t s_nc[kMaxLevel][kUnits];
    __shared__ uint32_t s_cnt[kMaxLevel];               // such nodes of a level
    if (in.m->ncells == 0) return;
    const int t = threadIdx.x;
    // the runs [r0, r1) of the workgroup
    uint32_t r1 = in.nedges, e0 = 0, e1 = 0;            // [e0, e1): the thread's unit
    if (kAll) {
        if (t < kUnits) {
            e0 = unit_begin(in, depth, (uint32_t)t);
            e1 = unit_begin(in, depth, (uint32_t)t + 1u);
        }
    } else {
        const uint32_t r0 = unit_begin(in, depth + 1u, blockIdx.x);
        r1 = unit_begin(in, depth + 1u, blockIdx.x + 1u);
        // r0 begins the lesser unit r0 >> (kUnitLog * depth)
        if (t < kUnits) {
            const uint32_t u = (r0 >> (kUnitLog * depth)) + (uint32_t)t;
            e0 = unit_begin(in, depth, u);
            e1 = unit_begin(in, depth, u + 1u);
        }
    }
    const int64_t range_end = run_begin(in, r1);
    if (t < kMaxLevel) s_cnt[t] = 0;
    __syncthreads();
    // nothing reaches beyond the last unit, and what reaches beyond the larger one is not
    // done here
    if (e1 > e0 && e1 < r1) {
        // the nodes holding both the unit's last particle and the next one: those of the
        // levels above the one where the two part and above the last one's leaf
        const RunEdge &a = in.edges[e0], &b = in.edges[e1];
        const int top = min((int)b.split, (int)in.lam[b.x - 1]);
        uint32_t c[kMaxLevel], ch[kMaxLevel], nc[kMaxLevel], f[kMaxLevel], cnt[kMaxLevel];
#pragma unroll
        for (int lev = 0; lev < kMaxLevel; ++lev) {
            c[lev] = 0;
            if (lev >= top) continue;
            const uint32_t e = b.c[lev];
            c[lev] = e > a.c[lev] ? in.m->level_offset[lev] + e : 0u;   // one past the last start
        }
#pragma unroll
        for (int lev = 0; lev < kMaxLevel; ++lev) {
            const uint32_t q = c[lev] ? c[lev] - 1u : 0u;
            f[lev] = cnt[lev] = ch[lev] = nc[lev] = 0;
            if (!c[lev]) continue;
            if (!kAll) {
                f[lev] = in.first[q];
                cnt[lev] = in.count[q];
            }
            ch[lev] = in.child[q];
            nc[lev] = in.nchild[q];
        }
#pragma unroll
        for (int lev = 0; lev < kMaxLevel; ++lev) {
            if (!c[lev] || (!kAll && (int64_t)f[lev] + cnt[lev] > range_end)) continue;
            const uint32_t i = atomicAdd(&s_cnt[lev], 1u);
            s_cell[lev][i] = c[lev] - 1u;
            s_ch[lev][i] = ch[lev];
            s_nc[lev][i] = (uint8_t)min(nc[lev], 8u);
        }
    }
    __syncthreads();
    TeamTerms &L = s_terms[t / kWave];
    const uint32_t team = (uint32_t)t / kTeam, team0 = (uint32_t)t / kWave * (kWave / kTeam);
    for (int lev = kMaxLevel - 1; lev >= 0; --lev) {
        const uint32_t count = s_cnt[lev];
        if (count == 0u) continue;          // uniform
        for (uint32_t i0 = 0; i0 + team0 < count; i0 += kTeams) {
            const uint32_t i = i0 + team;
            const bool has = i < count;
            node_from_memory<kBox>(L, has ? s_cell[lev][i] : 0u, has ? s_ch[lev][i] : 0u,
                                   has ? s_nc[lev][i] : 0u, c_com, c_S, box);
        }
        __syncthreads();
    }
    for (int i = t; i < kMaxLevel * kUnits; i += kThreads) {
        const int lev = i / kUnits, q = i % kUnits;
        if ((uint32_t)q >= s_cnt[lev]) continue;
        const uint32_t c = s_cell[lev][q];
        double m[kBox ? 16 : 10];
        load_moments<kBox>(c, c_com, c_S, box, m);
        moments_record<kBox>(c, in.first[c], lev, ro.c_cl[c], false, s_ch[lev][q], s_nc[lev][q], m,
                             ro);
    }
}

// The opening radii and walk records of every cell from its stored moments (the
// moments kernels write them as they go; this pass serves force calls whose
// theta or opening test differ from those the moments saw).  See cell_record.
__global__ void __launch_bounds__(kBlock)
rcrit_kernel(DevMisc *__restrict__ m, RecOut ro, const uint32_t *__restrict__ c_first,
             const uint32_t *__restrict__ c_count, const uint32_t *__restrict__ c_child,
             const uint32_t *__restrict__ c_nchild, const uint8_t *__restrict__ c_leaf,
             const double4 *__restrict__ c_com, const double *__restrict__ box)
{
    const uint32_t ncells = m->ncells;
    for (uint32_t c = blockIdx.x * kBlock + threadIdx.x; c < ncells; c += gridDim.x * kBlock) {
        const uint32_t f = c_first[c];
        const bool leaf = c_leaf[c] != 0;
        double bx[6];
        if (box) {
#pragma unroll
            for (int i = 0; i < 6; ++i) bx[i] = box[6 * (int64_t)c + i];
        }
        float s3[6];        // 3 S stays as it is in the record
#pragma unroll
        for (int q = 0; q < 6; ++q) s3[q] = ro.rec[c].s3[q];
        cell_record(c, f, ro.c_level[c], ro.c_cl[c], leaf, leaf ? f : c_child[c],
                    leaf ? c_count[c] : c_nchild[c], c_com[c], s3, box ? bx : nullptr,
                    box ? bx + 3 : nullptr, ro);
    }
}

}  // namespace

// ---------------------------------------------------------------------------

hipError_t launch_cluster_ids(bh_ctx *c)
{
    hipLaunchKernelGGL(cluster_ids_kernel, dim3((unsigned)c->nchunks), dim3(kBlock), 0, c->stream,
                       c->chunks, c->pcl);
    BH_LAUNCH_CHECK();
    return hipSuccess;
}

// whether the keys kernel makes the clusters' cubes
static bool domain_with_keys(const bh_ctx *c) { return c->max_cluster <= kKeysChunks * kChunk; }

// the chunks' boxes and, unless the keys kernel makes them, the clusters' cubes
hipError_t launch_domain(bh_ctx *c, const double *pos_aos)
{
    if (!pos_aos && c->box_ready) {
        // the partials of the held positions came with the step's drift
        c->box_ready = false;
    } else if (pos_aos)
        hipLaunchKernelGGL(bbox_kernel<AosSrc>, dim3((unsigned)c->nchunks), dim3(kBlock), 0,
                           c->stream, AosSrc{pos_aos}, c->chunks, c->bb_part, c->misc);
    else
        hipLaunchKernelGGL(bbox_kernel<P4Src>, dim3((unsigned)c->nchunks), dim3(kBlock), 0,
                           c->stream, P4Src{c->p4[c->cur]}, c->chunks, c->bb_part, c->misc);
    BH_LAUNCH_CHECK();
    if (!domain_with_keys(c)) {
        hipLaunchKernelGGL(domain_kernel, dim3((unsigned)c->K), dim3(kBlock), 0, c->stream,
                           c->bb_part, c->clus, c->dom);
        BH_LAUNCH_CHECK();
    }
    return hipSuccess;
}

hipError_t launch_keys(bh_ctx *c, const double *pos_aos)
{
    const uint32_t sub = c->nbuckets > 0 ? (uint32_t)sort_sub(c) : 0u;
    const uint32_t held = sort_sub(c) > 0 ? 1u : 0u;
    const double *part = domain_with_keys(c) ? c->bb_part : nullptr;
    if (pos_aos)
        hipLaunchKernelGGL(keys_kernel<AosSrc>, dim3((unsigned)c->nchunks), dim3(kBlock), 0,
                           c->stream, AosSrc{pos_aos}, c->chunks, part, c->dom, nullptr, (uint32_t)c->n,
                           c->key[0], c->val[0], 0u, c->clus, sub, sort_candidates(c), c->misc);
    else
        // a rebuild: held-order pairs for the bucket sort, caller-order pairs for
        // the radix sort
        hipLaunchKernelGGL(keys_kernel<P4Src>, dim3((unsigned)c->nchunks), dim3(kBlock), 0,
                           c->stream, P4Src{c->p4[c->cur]}, c->chunks, part, c->dom, c->pid[c->cur],
                           (uint32_t)c->n, c->key[0], c->val[0], held, c->clus, sub,
                           sort_candidates(c), c->misc);
    BH_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_reorder_from_caller(bh_ctx *c, const double *pos_aos, const double *mass,
                                      const double *vel, const uint32_t *perm)
{
    hipLaunchKernelGGL(reorder_from_caller_kernel, dim3(grid_for(c->n, kBlock)), dim3(kBlock), 0,
                       c->stream, pos_aos, mass, vel, perm, c->n, c->p4[c->cur], c->v4[c->cur],
                       c->pid[c->cur], c->misc);
    BH_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_reorder(bh_ctx *c, const uint32_t *perm)
{
    const int s = c->cur, d = c->cur ^ 1;
    hipLaunchKernelGGL(reorder_kernel, dim3(grid_for(c->n, kBlock)), dim3(kBlock), 0, c->stream,
                       c->p4[s], c->v4[s], c->pid[s], perm, c->n, c->p4[d], c->v4[d], c->pid[d],
                       c->misc);
    BH_LAUNCH_CHECK();
    c->cur = d;
    return hipSuccess;
}

namespace {

// the runs' edges, behind the level rows
RunEdge *run_edges(const bh_ctx *c)
{
    return reinterpret_cast<RunEdge *>(c->blk + level_rows_words(c->n));
}

}  // namespace

int64_t run_edge_words(int64_t n)
{
    return (int64_t)(sizeof(RunEdge) / sizeof(uint32_t)) * most_runs(n);
}

hipError_t launch_tree(bh_ctx *c)
{
    const int64_t n = c->n;
    const int nblk = grid_for(n, kTreeTile);
    uint32_t *blk = c->blk;                       // [kLevels + 1][nblk]
    uint32_t *tot = c->blk + (int64_t)(kLevels + 1) * nblk;
    const int H = c->max_nleaf;
    const size_t lds = (size_t)((kTreeTile + 2 * H + 15) & ~15) + (size_t)kTreeTile * H;
    hipLaunchKernelGGL(split_leaf_kernel, dim3(nblk), dim3(kTreeTile), lds, c->stream, c->key[0],
                       c->pcl, n, H, c->clus, c->split, c->lam, c->gflag, blk, nblk, c->misc);
    BH_LAUNCH_CHECK();
    const bool scan = nblk <= kEmitTiles;
    if (!scan) {
        hipLaunchKernelGGL(scan_levels_kernel, dim3(kLevels + 1), dim3(kScanLevelsBlock), 0,
                           c->stream, blk, nblk, tot, c->misc, c->cap_c);
        BH_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(scan ? emit_cells_kernel<true> : emit_cells_kernel<false>, dim3(nblk),
                       dim3(kTreeTile), 0, c->stream, c->split, c->lam, n, blk, nblk, c->misc,
                       c->cap_c, c->c_first, c->c_level, c->c_leaf, c->c_parent, c->c_child,
                       c->c_end, c->c_nchild, c->pcl, c->c_cl, run_edges(c),
                       run_tiles_log(c->n, c->run_leaf));
    BH_LAUNCH_CHECK();
    int g = grid_for(c->cap_c, kBlock);
    if (g > kFixedGrid) g = kFixedGrid;
    hipLaunchKernelGGL(cell_finish_kernel, dim3(g), dim3(kBlock), 0, c->stream, c->misc, c->pcl,
                       c->clus, c->c_first, c->c_end, c->c_leaf, c->c_level, c->c_parent,
                       c->c_child, c->c_count, c->c_nchild, c->gflag, n);
    BH_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_groups(bh_ctx *c)
{
    return compact_flags(c, c->gflag, c->n, c->g_first, &c->misc->ngroups, walk_order(c, false),
                         c->misc->upto, true);
}

hipError_t launch_group_boxes(bh_ctx *c)
{
    int g = grid_for(c->n, kBlock / 16);
    if (g > kFixedGrid) g = kFixedGrid;
    hipLaunchKernelGGL(group_boxes_kernel, dim3(g), dim3(kBlock), 0, c->stream, c->g_first, c->misc,
                       c->n, c->p4[c->cur], c->pcl, c->g_count, c->g_centre, c->g_half);
    BH_LAUNCH_CHECK();
    return hipSuccess;
}

// The leaves and nodes within runs, then the nodes across runs: of up to kSpanUnits runs
// in one workgroup, of more first in units of about 64 runs, a workgroup each, and then
// across those.  The time is the chain of levels, not the bytes (a level's barrier, its
// LDS or L2 reads, two divisions): leaves and nodes in one launch per level or group of
// levels took 28, 89, 110 and 412 us at 1500, 240K and 2^20 particles and for 512 clusters
// of 1024 to 65,536, this 19, 43, 96 and 354.  Units beginning at any multiple of their
// size, not between large cells: 19, 61, 103, 386.  The sizes of the runs and which systems
// one workgroup holds whole: moment_rules.h.
// kSpanUnits: as many as the lists of their nodes leave LDS for (builds of 300,000 and
// 500,000 particles 232 and 261 us, with 256 units, so one launch more, 255 and 286).
constexpr int kSpanUnits = 512;

template <bool kBox, int kThreads, int kCap, int kTiles>
void runs_launch(bh_ctx *c, uint32_t runs, const CellIn &in, double *box, const RecOut &ro)
{
    hipLaunchKernelGGL((run_moments_kernel<kBox, kThreads, kCap, 1, kTiles>), dim3(runs),
                       dim3(kThreads), 0, c->stream, in, c->c_com, c->c_S, box, ro);
}

template <bool kBox>
hipError_t moments_launches(bh_ctx *c, double *box)
{
    // every cell's opening radius and walk record are written with its moments
    const RecOut ro{c->clus, c->dom, c->c_level, c->c_cl, c->key[0], c->c_rcrit2, c->c_rec, c->c_geo};
    const int tiles_log = run_tiles_log(c->n, c->run_leaf);
    const uint32_t runs = (uint32_t)grid_for(c->n, kTreeTile << tiles_log);
    const CellIn in{c->misc, run_edges(c), runs, c->n, c->lam, c->c_leaf, c->c_first, c->c_count,
                    c->c_child, c->c_nchild, c->p4[c->cur]};
    // (with boxes, the moments of a whole system need more LDS than there is)
    if (!kBox && one_workgroup(c->n, c->K, c->run_leaf)) {
        hipLaunchKernelGGL((run_moments_kernel<false, 1024, 1279, 16, 1>), dim3(1), dim3(1024), 0,
                           c->stream, in, c->c_com, c->c_S, box, ro);
        BH_LAUNCH_CHECK();
        c->rec_fresh = true;
        return hipSuccess;
    }
    if (tiles_log == 0) runs_launch<kBox, 256, kBox ? 495 : 463, 1>(c, runs, in, box, ro);
    else if (tiles_log == 1) runs_launch<kBox, 256, kBox ? 191 : 255, 2>(c, runs, in, box, ro);
    else if (c->n <= (kBox ? kWideRunsBox : kWideRuns)) runs_launch<kBox, 512, 511, 4>(c, runs, in, box, ro);
    else runs_launch<kBox, 256, kBox ? 303 : 463, 4>(c, runs, in, box, ro);
    BH_LAUNCH_CHECK();
    if (runs > 1) {
        uint32_t depth = 0, units = runs;
        for (; units > kSpanUnits; ++depth) {
            units = (uint32_t)grid_for(units, 1 << kUnitLog);
            hipLaunchKernelGGL((span_moments_kernel<kBox, 80, 512, false>), dim3(units), dim3(512), 0,
                               c->stream, in, depth, c->c_com, c->c_S, box, ro);
            BH_LAUNCH_CHECK();
        }
        hipLaunchKernelGGL((span_moments_kernel<kBox, kSpanUnits, 1024, true>), dim3(1), dim3(1024), 0,
                           c->stream, in, depth, c->c_com, c->c_S, box, ro);
        BH_LAUNCH_CHECK();
    }
    c->rec_fresh = true;
    return hipSuccess;
}

hipError_t launch_moments(bh_ctx *c, bool boxes)
{
    if (boxes) return moments_launches<true>(c, c->c_box);
    return moments_launches<false>(c, nullptr);
}

hipError_t launch_rcrit(bh_ctx *c)
{
    // the moments pass wrote the records with the current table already
    if (c->rec_fresh) return hipSuccess;
    int g = grid_for(c->cap_c, kBlock);
    if (g > kFixedGrid) g = kFixedGrid;
    const RecOut ro{c->clus, c->dom, c->c_level, c->c_cl, c->key[0], c->c_rcrit2, c->c_rec, c->c_geo};
    hipLaunchKernelGGL(rcrit_kernel, dim3(g), dim3(kBlock), 0, c->stream, c->misc, ro, c->c_first,
                       c->c_count, c->c_child, c->c_nchild, c->c_leaf, c->c_com,
                       c->refitted ? c->c_box : nullptr);
    BH_LAUNCH_CHECK();
    c->rec_fresh = true;
    return hipSuccess;
}

}  // namespace bh
