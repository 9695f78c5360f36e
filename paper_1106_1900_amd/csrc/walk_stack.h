// walk_stack.h - the walk's stack of pending cells (see walk.hip).  It is written in the
// wavefront primitives of bh_internal.h, included before it, so that the same source also
// runs on the CPU over 64 emulated lanes (tests/walk_stack_host.cpp).
#pragma once

namespace bh {
namespace {

constexpr int kLdsStack = 384;
constexpr int kSpillPerWave = 1280;
// Entries the stack can hold: kSpillPerWave, and what a push that spills leaves in LDS.
constexpr int kStackKept = kLdsStack - kWave;
constexpr int kStackCap = kSpillPerWave + kStackKept;
// A pop of w cells pushes at most 8 w, so it takes 64 only while 7 * 64 more entries fit
// and, below that, as many as fit seven times (at least one) over a reserve: by single
// cells, a cell's whole subtree takes at most 7 entries a level.
constexpr int kStackReserve = 7 * kMaxLevel + 8;

// The stack of pending cells: its top entries in LDS, `base` entries below them in
// device memory.
struct CellStack {
    uint32_t *s;                // LDS, kLdsStack entries
    volatile uint32_t *spill;   // kSpillPerWave entries
    int top;                    // entries in LDS
    int base;

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
    // All but the top kStackKept entries of the stack and the push go to device memory.
    __device__ bool push_spilling(bool node, int at, uint32_t last, uint32_t c1, int total)
    {
        const int lane = lane_id();
        if (base + top + total > kStackCap) return false;
        const int cut = top + total - kStackKept;       // > 0; at most kSpillPerWave - base
        for (int i = lane; i < min(top, cut); i += kWave) spill[base + i] = s[i];
        wave_sync();
        for (int i = cut; i < top; i += kWave) {
            const uint32_t v = i + lane < top ? s[i + lane] : 0u;
            wave_sync();
            if (i + lane < top) s[i - cut + lane] = v;
            wave_sync();
        }
        if (node) {
            for (uint32_t r = 0; r <= c1; ++r) {
                const int i = at + (int)r;
                if (i < cut) spill[base + i] = last - r;
                else s[i - cut] = last - r;
            }
        }
        base += cut;
        top = kStackKept;
        sync();
        return true;
    }

    // up to 128 entries back from device memory, below the fewer than 64 in LDS
    __device__ void refill()
    {
        const int lane = lane_id();
        const int d = min(base, 2 * kWave);
        const uint32_t v = lane < top ? s[lane] : 0u;
        wave_sync();
        if (lane < top) s[d + lane] = v;
        for (int i = lane; i < d; i += kWave) s[i] = spill[base - d + i];
        base -= d;
        top += d;
        sync();
    }
};

}  // namespace
}  // namespace bh
