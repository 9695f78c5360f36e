"""CPU tests of the walk's hand-out rules (walk_handout.h): which groups whole workgroups
walk.  Groups of up to 16 particles and those of small clusters have short lists, and a
workgroup for each of them leaves the others waiting; where most groups are large, teams
would walk the tree for each of them in several rounds."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1106_1900_amd", "csrc")
SRC = r"""
#define __host__
#define __device__
#include <cstdio>
#include <cstdlib>
#include "walk_handout.h"
using namespace bh;
int main(int argc, char **a)
{
    // depth theta mac waves per workgroup, then pairs: groups, size (of clusters of 10,000)
    uint32_t upto[kGroupClasses] = {}, n = 0;
    for (int i = 6; i + 1 < argc; i += 2) {
        const uint32_t count = std::atoi(a[i]);
        for (int c = 0; c < group_class(std::atoi(a[i + 1]), 10000u); ++c) upto[c] += count;
        n += count;
    }
    const int waves = std::atoi(a[4]), per = std::atoi(a[5]);
    std::printf("%u", team_groups(upto, n, waves, waves / per,
                                  short_lists(std::atoi(a[1]), std::atof(a[2]), std::atoi(a[3]))));
}
"""
CLASSES = r"""
#define __host__
#define __device__
#include <cstdio>
#include <cstdlib>
#include "walk_handout.h"
int main(int, char **a) { std::printf("%d", bh::group_class(std::atoi(a[1]), std::atoi(a[2]))); }
"""


def _compile(d, name, text):
    (d / (name + ".cpp")).write_text(text)
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(d / (name + ".cpp")), "-o",
                           str(d / name)])

    def run(*args):
        out = subprocess.run([str(d / name), *map(str, args)], capture_output=True, text=True,
                             check=True)
        return int(out.stdout)
    return run


@pytest.fixture(scope="module")
def teams(tmp_path_factory):
    run = _compile(tmp_path_factory.mktemp("handout"), "teams", SRC)

    def of(groups, depth=10, theta=0.75, mac=0, waves=4096, per=4):
        return run(depth, theta, mac, waves, per, *[x for g in groups for x in g])
    return of


@pytest.mark.parametrize("size,cluster,same", [
    (1, 400, 8), (8, 400, 1), (9, 400, 16), (17, 321, 32), (33, 400, 48), (49, 400, 64),
    (65, 400, 128), (64, 64, 1), (64, 320, 1), (2, 2, 1),
])
def test_classes(tmp_path, size, cluster, same):
    cls = _compile(tmp_path, "classes", CLASSES)
    assert cls(size, cluster) == cls(same, max(cluster, 321) if cluster > 320 else cluster)


@pytest.mark.parametrize("groups,want", [
    ([(1000, 1)], 0), ([(684, 16)], 0), ([(200, 16), (300, 17)], 300),
    ([(1024, 32)], 1024), ([(1025, 32)], 0), ([(1000, 32), (25, 33)], 25),
    ([(2500, 32), (60, 33)], 60), ([(2500, 32), (61, 33)], 0), ([(2500, 32), (61, 49)], 61),
    ([(6000, 32), (144, 49)], 144), ([(6000, 32), (145, 49)], 0), ([(6000, 32), (145, 65)], 145),
    ([(16000, 32), (384, 65)], 384), ([(16000, 32), (385, 65)], 0),
    # more of a class than there are workgroups: the next one, or none
    ([(1025, 49)], 0), ([(1025, 49), (3, 65)], 3), ([(2000, 20), (1024, 49)], 1024),
    ([(4000, 65)], 0),
])
def test_which_groups_teams_walk(teams, groups, want):
    assert teams(groups) == want


def test_wide_workgroups(teams):
    assert teams([(512, 32)], per=8) == 512
    assert teams([(513, 32), (2, 33)], per=8) == 2


@pytest.mark.parametrize("depth,theta,mac,want", [
    (4, 0.75, 0, 7), (6, 0.75, 0, 307), (4, 0.55, 0, 307), (4, 0.75, 1, 307),
])
def test_short_lists(teams, depth, theta, mac, want):
    assert teams([(300, 20), (7, 40)], depth, theta, mac) == want


OWN = r"""
#define __host__
#define __device__
#include <cstdio>
#include <cstdlib>
#include "walk_handout.h"
int main(int, char **a)
{
    std::printf("%d", bh::first_own_class(std::atoll(a[1]), 4096, std::atoll(a[2])));
}
"""


@pytest.mark.parametrize("ngroups,clusters,size", [
    (1, 1, 1), (16385, 1, 1), (32768, 1, 1), (32769, 1, 17), (98304, 1, 17), (75400, 300, 49),
    (32768, 300, 1), (50000, 100, 17), (49999, 100, 49),
])
def test_small_groups_stay_in_tree_order(tmp_path, ngroups, clusters, size):
    """With several groups per wavefront only the large ones are taken out of Morton order."""
    own = _compile(tmp_path, "own", OWN)
    cls = _compile(tmp_path, "classes", CLASSES)
    assert own(ngroups, clusters) == cls(size, 400)
