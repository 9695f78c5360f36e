// The walk's stack (csrc/walk_stack.h) on the CPU: 64 lanes as fibers that meet at every
// wavefront primitive, memory as plain arrays with guarded ends.  Between two primitives
// the lanes run one after the other, in lane order.
//
//   walk_stack_host childless        nodes without children among others push nothing
//   walk_stack_host tree B D         a full tree of B children a node and D levels: every
//                                    cell is popped once
//   walk_stack_host deep P           nodes of eight children down to level 20 for P pops,
//                                    then leaves: the stack holds them, each popped once
//
// Prints "ok" and the most cells pending, the most words in device memory and the narrowest
// pop while 64 cells were pending; exits with 1 and a message otherwise.
#include <ucontext.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

using std::max;
using std::min;

namespace bh {

constexpr int kMaxLevel = 20;
constexpr int kWave = 64;

namespace emu {

ucontext_t sched, lanes[kWave];
std::vector<char> stacks(kWave * (64 << 10));
std::function<void()> body;
int cur = 0;
bool done[kWave];
int ops[kWave];
uint64_t slot[2][kWave];
int phase[kWave];

void die(const char *msg)
{
    printf("failed: %s\n", msg);
    fflush(stdout);
    _Exit(1);
}

// every lane's value of a primitive; op names it
const uint64_t *meet(int op, uint64_t v)
{
    const int l = cur, ph = phase[l];
    phase[l] ^= 1;
    slot[ph][l] = v;
    ops[l] = op;
    swapcontext(&lanes[l], &sched);
    return slot[ph];
}

void entry()
{
    body();
    done[cur] = true;
    ops[cur] = -1;
    swapcontext(&lanes[cur], &sched);
}

// one call of f by all lanes
void run(const std::function<void()> &f)
{
    body = f;
    for (int l = 0; l < kWave; ++l) {
        getcontext(&lanes[l]);
        lanes[l].uc_stack.ss_sp = &stacks[(size_t)l * (64 << 10)];
        lanes[l].uc_stack.ss_size = 64 << 10;
        lanes[l].uc_link = &sched;
        makecontext(&lanes[l], (void (*)())entry, 0);
        done[l] = false;
        phase[l] = 0;
    }
    for (;;) {
        for (cur = 0; cur < kWave; ++cur) swapcontext(&sched, &lanes[cur]);
        for (int l = 1; l < kWave; ++l)
            if (ops[l] != ops[0]) die("lanes meet at different primitives");
        if (done[0]) return;
    }
}

}  // namespace emu

int lane_id() { return emu::cur; }

unsigned long long ballot(bool p)
{
    const uint64_t *v = emu::meet(1, p);
    unsigned long long m = 0;
    for (int l = 0; l < kWave; ++l) m |= (unsigned long long)(v[l] != 0) << l;
    return m;
}

int mask_rank(unsigned long long m) { return __builtin_popcountll(m & ((1ull << emu::cur) - 1)); }

void wave_sync() { emu::meet(2, 0); }

uint32_t wave_incl_scan_add(uint32_t x)
{
    const uint64_t *v = emu::meet(3, x);
    uint32_t s = 0;
    for (int l = 0; l <= emu::cur; ++l) s += (uint32_t)v[l];
    return s;
}

uint32_t lane_value(uint32_t x, int i) { return (uint32_t)emu::meet(4, x)[i]; }

}  // namespace bh

#define __device__
#define __forceinline__ inline
#define __popcll __builtin_popcountll
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#include "walk_stack.h"

using namespace bh;

namespace {

constexpr uint32_t kGuard = 0xa5a5a5a5u;
constexpr int kPad = 1024;
std::vector<uint32_t> lds(kLdsStack + 2 * kPad, kGuard), mem(kSpillPerWave + 2 * kPad, kGuard);
CellStack lane_stack[kWave];        // each lane's copy of the wavefront's registers

struct Node {
    uint32_t link, n;
    int level;
};
std::vector<Node> cells;
std::vector<uint8_t> popped;
int64_t pending = 0;                // cells
int64_t deepest = 0;
int spilled = 0, narrowest = kWave;

void check()
{
    for (int i = 0; i < kPad; ++i)
        if (lds[i] != kGuard || lds[kPad + kLdsStack + i] != kGuard || mem[i] != kGuard ||
            mem[kPad + kSpillPerWave + i] != kGuard)
            emu::die("write outside the stack");
    for (int l = 1; l < kWave; ++l)
        if (lane_stack[l].top != lane_stack[0].top || lane_stack[l].base != lane_stack[0].base)
            emu::die("lanes hold different stacks");
    const int top = lane_stack[0].top, base = lane_stack[0].base;
    if (top < 0 || top > kLdsStack || base < 0 || base > kSpillPerWave) emu::die("stack out of range");
    deepest = max(deepest, pending);
    spilled = max(spilled, base);
}

void start(uint32_t root)
{
    for (int l = 0; l < kWave; ++l)
        lane_stack[l] = CellStack{lds.data() + kPad, mem.data() + kPad, 1, 0};
    lds[kPad] = root;
    pending = 1;
}

// the cells of a pop, one per lane
int pop(uint32_t *cell)
{
    int got[kWave];
    emu::run([&] {
        const int l = lane_id();
        got[l] = lane_stack[l].pop(cell[l]);
    });
    for (int l = 1; l < kWave; ++l)
        if (got[l] != got[0]) emu::die("lanes popped different numbers");
    if (got[0] < 1 || got[0] > kWave) emu::die("nothing popped from a stack that holds cells");
    if (pending >= kWave) narrowest = min(narrowest, got[0]);
    pending -= got[0];
    check();
    return got[0];
}

void push(const bool *node, const Node *v)
{
    bool full = false;
    emu::run([&] {
        const int l = lane_id();
        if (!lane_stack[l].push(node[l], v[l].link, v[l].n)) full = true;
    });
    if (full) emu::die("stack full");
    for (int l = 0; l < kWave; ++l)
        if (node[l]) pending += min(v[l].n, 8u);
    check();
}

// pops until nothing is pending; open(cell) gives the children to push (n = 0: a leaf)
template <class Open>
void walk(Open open)
{
    while (pending > 0) {
        uint32_t cell[kWave];
        const int got = pop(cell);
        bool node[kWave] = {};
        Node v[kWave] = {};
        for (int l = 0; l < got; ++l) {
            if (cell[l] >= cells.size()) emu::die("a cell that was never pushed");
            if (popped[cell[l]]++) emu::die("a cell popped twice");
            v[l] = open(cell[l]);
            node[l] = v[l].n > 0;
        }
        push(node, v);
    }
    if (lane_stack[0].top || lane_stack[0].base) emu::die("entries left");
    for (uint8_t p : popped)
        if (p != 1) emu::die("a cell lost");
}

// appends n cells of a level
uint32_t add(uint32_t n, int level)
{
    const uint32_t first = (uint32_t)cells.size();
    for (uint32_t i = 0; i < n; ++i) cells.push_back({0, 0, level});
    popped.resize(cells.size());
    return first;
}

void childless()
{
    // nodes of 0 to 8 children, at every fill of the stack's LDS part
    for (int fill = 1; fill <= kLdsStack; fill += 13) {
        start(0);
        for (int i = 0; i < fill; ++i) lds[kPad + i] = 1000000u + (uint32_t)i;
        for (int l = 0; l < kWave; ++l) lane_stack[l].top = fill;
        pending = fill;
        bool node[kWave];
        Node v[kWave];
        int want = fill;
        for (int l = 0; l < kWave; ++l) {
            node[l] = l % 3 != 0;
            v[l] = Node{100u * (uint32_t)l, (uint32_t)((l / 3) % 9), 0};
            if (node[l]) want += (int)v[l].n;
        }
        push(node, v);
        std::vector<uint32_t> got, exp;
        for (int i = fill; i-- > 0;) exp.push_back(1000000u + (uint32_t)i);
        std::vector<uint32_t> kids;
        for (int l = kWave; l-- > 0;)
            for (uint32_t c = 0; node[l] && c < v[l].n; ++c) kids.push_back(v[l].link + c);
        exp.insert(exp.begin(), kids.begin(), kids.end());
        if ((int)exp.size() != want) emu::die("model");
        while (pending > 0) {
            uint32_t cell[kWave];
            const int n = pop(cell);
            got.insert(got.end(), cell, cell + n);
        }
        if (got != exp) emu::die("cells lost, invented or out of order");
    }
}

void tree(uint32_t b, int depth)
{
    // level by level, as the cell array is laid out
    uint32_t lo = add(1, 0), hi = lo + 1;
    for (int lev = 1; lev < depth; ++lev) {
        for (uint32_t c = lo; c < hi; ++c) {
            cells[c].n = b;
            const uint32_t first = add(b, lev);
            cells[c].link = first;
        }
        lo = hi;
        hi = (uint32_t)cells.size();
    }
    start(0);
    walk([](uint32_t c) { return cells[c]; });
}

void deep(int pops)
{
    add(1, 0);
    start(0);
    int left = pops * kWave;
    walk([&](uint32_t c) {
        Node v{0, 0, 0};
        if (cells[c].level < kMaxLevel && left-- > 0) {
            v.n = 8;
            v.link = add(8, cells[c].level + 1);
        }
        return v;
    });
}

}  // namespace

int main(int argc, char **argv)
{
    if (argc > 1 && !strcmp(argv[1], "childless")) childless();
    else if (argc > 3 && !strcmp(argv[1], "tree")) tree((uint32_t)atoi(argv[2]), atoi(argv[3]));
    else if (argc > 2 && !strcmp(argv[1], "deep")) deep(atoi(argv[2]));
    else return 2;
    printf("ok %d %d %d\n", (int)deepest, spilled, narrowest);
    return 0;
}
