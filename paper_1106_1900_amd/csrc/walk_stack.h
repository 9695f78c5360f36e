// walk_stack.h - the walk's stack of pending cells (see walk.hip).  It is written in the
// wavefront primitives of bh_internal.h, included before it, so that the same source also
// runs on the CPU over 64 emulated lanes (tests/walk_stack_host.cpp).
#pragma once

namespace bh {
namespace {

constexpr int kLdsStack = 384;
constexpr int kSpillPerWave = 1280;
// Cells and ranges the stack can hold: kSpillPerWave, and what a push that spills leaves
// in LDS.
constexpr int kStackKept = kLdsStack - kWave;
constexpr int kStackCap = kSpillPerWave + kStackKept;
// A pop of w cells pushes at most 8 w, so it takes 64 only while 7 * 64 more entries fit
// and, below that, as many as fit seven times (at least one) over a reserve: by single
// cells, a cell's whole subtree takes at most 7 entries a level, and so do those of a
// range that comes back to an empty LDS part.
constexpr int kStackReserve = 7 * kMaxLevel + 16;
constexpr int kRefill = 256;    // most cells that come back at once

// The stack of pending cells: the top ones in LDS, a word each, those below in device
// memory as ranges of up to 8 consecutive cells (a node's children, mostly), packed in
// 32 bits as first cell << 3 | count - 1.  So the stack is about as deep as its nodes are
// many, and pops take 64 cells wherever 64 are pending but in trees that none of the
// models comes near (20 levels of nodes, all with eight children and all opened).  With a
// word per cell in device memory too, walks that open many cells filled it and popped
// fewer and fewer cells at a time: 200,000 particles of a Hernquist sphere at theta = 0.2
// by the minimum distance (leaves of 8) 21.6 ms, 7.9 so, 262,144 of a galaxy at 0.2 8.7
// ms, 5.2 so.
struct CellStack {
    uint32_t *s;                // LDS, kLdsStack entries
    volatile uint32_t *spill;   // kSpillPerWave entries
    int top;                    // entries in LDS
    int base;                   // ranges in device memory

    // stores to device memory must have landed before another lane reads them
    __device__ void sync() const
    {
        __builtin_amdgcn_s_waitcnt(0);
        wave_sync();
    }

    // Up to 64 cells from the top, one per lane; returns how many.
    __device__ __forceinline__ int pop(uint32_t &cell)
    {
        const int lane = lane_id();
        if (__builtin_expect(top < kWave && base > 0, 0)) refill();
        const int room = kStackCap - kStackReserve - (base + top);
        int m = top < kWave ? top : kWave;
        if (__builtin_expect(room < 7 * kWave, 0)) m = min(m, max(1, room / 7));
        cell = lane < m ? s[top - 1 - lane] : 0u;
        top -= m;
        return m;
    }

    // The children of each lane's opened cell (record fields link and info, see WalkCell):
    // [link, link + info) of a node, at most 8; none of a leaf, nor if info = 0, which only
    // a record of an inconsistent tree holds.  The first lane's children lie deepest, a
    // node's first child on top of its others.
    // Every lane stores eight entries, those past its own children in the places of the
    // lanes above: the stores are issued from the eighth entry down to the first (they are
    // volatile, and a wavefront's LDS instructions execute in order), so each entry's
    // last store is its owner's.  Returns false if the stack is full (never).
    __device__ __forceinline__ bool push(bool open, uint32_t link, uint32_t info)
    {
        const bool node = open && (int32_t)info > 0;
        const uint32_t n = min(info, 8u);
        const unsigned long long bn = ballot(node);
        if (bn == 0ull) return true;
        const uint32_t c1 = node ? n - 1u : 0u;
        const unsigned long long b0 = ballot((c1 & 1u) != 0u), b1 = ballot((c1 & 2u) != 0u),
                                 b2 = ballot((c1 & 4u) != 0u);
        const int total = __popcll(bn) + __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
        const int at = top + mask_rank(bn) + mask_rank(b0) + 2 * mask_rank(b1) + 4 * mask_rank(b2);
        const uint32_t last = link + c1;
        if (__builtin_expect(top + total + 7 <= kLdsStack, 1)) {
            if (node) {
                // (as LDS by its type: volatile accesses keep the type they are given)
                using LdsWord = volatile __attribute__((address_space(3))) uint32_t;
                LdsWord *q = (LdsWord *)(s + at);
#pragma unroll
                for (int r = 7; r >= 0; --r) q[r] = last - (uint32_t)r;
            }
            top += total;
            wave_sync();
            return true;
        }
        return push_spilling(node, at, last, c1, total);
    }

private:
    // All but the top kStackKept cells of the stack and the push go to device memory.
    __device__ bool push_spilling(bool node, int at, uint32_t last, uint32_t c1, int total)
    {
        const int lane = lane_id();
        if (base + top + total > kStackCap) return false;
        const int cut = top + total - kStackKept;       // > 0; at most kSpillPerWave - base
        // the cells held, 64 at a time, by runs of descending numbers, eight to a range
        const int old = min(top, cut);
        for (int i = 0; i < old; i += kWave) {
            const int m = min(old - i, kWave);
            const uint32_t v = lane < m ? s[i + lane] : 0u;
            const uint32_t below = lane > 0 && lane < m ? s[i + lane - 1] : 0u;
            const unsigned long long runs = ballot(lane < m && (lane == 0 || v + 1u != below));
            const int in_run = __builtin_clzll((runs << (kWave - 1 - lane)) | 1ull);
            const bool first = lane < m && (in_run & 7) == 0;
            const unsigned long long b = ballot(first);
            if (first) {
                const unsigned long long next = (b >> lane) >> 1;
                const uint32_t c = next ? (uint32_t)__builtin_ctzll(next) : (uint32_t)(m - 1 - lane);
                spill[base + mask_rank(b)] = ((v - c) << 3) | c;
            }
            base += __popcll(b);
        }
        wave_sync();
        for (int i = cut; i < top; i += kWave) {
            const uint32_t v = i + lane < top ? s[i + lane] : 0u;
            wave_sync();
            if (i + lane < top) s[i - cut + lane] = v;
            wave_sync();
        }
        // the push: of a node's children those below the cut, then the others
        const int deep = node ? min((int)c1 + 1, max(0, cut - at)) : 0;
        const unsigned long long b = ballot(deep > 0);
        if (deep > 0) spill[base + mask_rank(b)] = ((last - (uint32_t)(deep - 1)) << 3) | (uint32_t)(deep - 1);
        base += __popcll(b);
        if (node)
            for (int r = deep; r <= (int)c1; ++r) s[at + r - cut] = last - (uint32_t)r;
        top = kStackKept;
        sync();
        return true;
    }

    // Ranges back from device memory, below the fewer than 64 cells in LDS: up to kRefill
    // cells, and no more than leave the next pop its full width.
    __device__ void refill()
    {
        const int lane = lane_id();
        const int m = min(base, kWave);
        const uint32_t w = lane < m ? spill[base - 1 - lane] : 0u;
        const int n = lane < m ? (int)(w & 7u) + 1 : 0;
        const int incl = (int)wave_incl_scan_add((uint32_t)n);
        const int room = kStackCap - kStackReserve - 7 * kWave - (base + top);
        const bool take = lane < m && incl <= kRefill && (incl - (lane + 1) <= room || (lane == 0 && top == 0));
        const int words = __popcll(ballot(take));       // the first lanes
        if (words == 0) return;
        const int cells = (int)lane_value((uint32_t)incl, words - 1);
        const uint32_t v = lane < top ? s[lane] : 0u;
        wave_sync();
        if (lane < top) s[cells + lane] = v;
        if (take)
            for (int r = 0; r < n; ++r) s[cells - incl + r] = (w >> 3) + (uint32_t)(n - 1 - r);
        base -= words;
        top += cells;
        sync();
    }
};

}  // namespace
}  // namespace bh
