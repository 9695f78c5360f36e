"""CPU tests of the walk's hand-out rules (walk_handout.h): which groups whole workgroups
walk.  Groups of up to 16 particles and those of small clusters have short lists, and a
workgroup for each of them leaves the others waiting."""

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
int main(int, char **a)
{
    std::printf("%d %d", bh::group_class(std::atoi(a[1]), std::atoi(a[2])),
                bh::team_class(std::atoi(a[3]), std::atoi(a[4])));
}
"""


@pytest.fixture(scope="module")
def by_team(tmp_path_factory):
    d = tmp_path_factory.mktemp("handout")
    (d / "rules.cpp").write_text(SRC)
    exe = str(d / "rules")
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(d / "rules.cpp"), "-o", exe])

    def run(size, cluster, ngroups, waves=4096):
        out = subprocess.run([exe, *map(str, (size, cluster, ngroups, waves))],
                             capture_output=True, text=True, check=True).stdout.split()
        cls, least = map(int, out)
        return least > 0 and cls >= least
    return run


@pytest.mark.parametrize("size,cluster,ngroups,team", [
    (1, 1000, 1000, False), (8, 1000, 100, False), (16, 3000, 684, False), (17, 3000, 684, True),
    (64, 4096, 276, True), (2, 2, 1000, False), (64, 64, 500, False), (64, 320, 10, False),
    (64, 321, 10, True),
    (32, 9000, 1025, False), (33, 9000, 1025, True), (33, 9000, 2560, True), (33, 9000, 2561, False),
    (49, 60000, 6144, True), (49, 60000, 6145, False), (65, 60000, 16384, True),
    (128, 200000, 16385, False),
])
def test_which_groups_teams_walk(by_team, size, cluster, ngroups, team):
    assert by_team(size, cluster, ngroups) == team
