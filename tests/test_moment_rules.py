"""CPU tests of the rules by which the moments are split (moment_rules.h): small leaves take
short runs, whose cells fit on chip, and the table of the runs' edges has room for them."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1106_1900_amd", "csrc")
SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "moment_rules.h"
using namespace bh;
int main(int argc, char **a)
{
    if (argc > 3) {
        const int64_t n = std::atoll(a[1]), k = std::atoll(a[2]);
        const int leaf = run_leaf(n, k, std::atoi(a[3]));
        std::printf("%d %d %d", leaf, 1 << run_tiles_log(n, leaf), one_workgroup(n, k, leaf));
        return 0;
    }
    // every run of every size has its edge, also in buffers made for more particles
    int64_t most = 0;
    for (int64_t n = 1; n < 3000000; n += n < 300000 ? 1 : 97) {
        if (most_runs(n) < most) return 1;
        most = most_runs(n);
        for (int leaf = 1; leaf <= 64; ++leaf) {
            const int64_t tile = kRunTile << run_tiles_log(n, leaf);
            if ((n + tile - 1) / tile > most) return 2;
            if (one_workgroup(n, 1, leaf) && (n + kRunTile - 1) / kRunTile > 16) return 3;
        }
    }
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("moments")
    (d / "rules.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, str(d / "rules.cpp"), "-o",
                           str(d / "rules")])
    return str(d / "rules")


@pytest.mark.parametrize("n,k,leaf,tiles,one", [
    (293, 1, 1, 4, True), (294, 1, 1, 1, True), (4096, 1, 16, 4, True), (4097, 1, 16, 4, False),
    (4096, 1, 8, 1, False), (2500, 1, 8, 1, True), (881, 1, 8, 4, True), (882, 1, 8, 1, True), (4096, 1, 1, 1, False),
    (131072, 1, 13, 1, False), (131073, 1, 13, 4, False), (1 << 19, 1, 8, 4, False),
    ((1 << 19) + 1, 1, 8, 2, False), (131073, 1, 2, 2, False), (1 << 22, 1, 14, 4, False),
    (2000, 1000, 16, 1, False), (1000000, 500000, 16, 2, False), (1000000, 10000, 16, 4, False),
])
def test_runs_and_workgroups(exe, n, k, leaf, tiles, one):
    out = subprocess.run([exe, str(n), str(k), str(leaf)], capture_output=True, text=True, check=True)
    assert out.stdout.split()[1:] == [str(tiles), str(int(one))]


def test_edges_have_room(exe):
    subprocess.run([exe], check=True)
