"""CPU tests of the rule that chooses the sort (sort_rules.h): thousands of tiny clusters
take the radix sort, and whatever takes buckets has at most 256 of them per cluster."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1106_1900_amd", "csrc")
SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "sort_rules.h"
int main(int, char **a)
{
    std::printf("%d", bh::sort_rule(std::atoll(a[1]), std::atoll(a[2]), std::atoll(a[3])));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rule.cpp").write_text(SRC)
    exe = str(d / "rule")
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(d / "rule.cpp"), "-o", exe])

    def run(sizes):
        chunks = [-(-n // 4096) for n in sizes]
        args = (sum(sizes), sum(chunks), max(sizes))
        out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, check=True)
        sub = int(out.stdout)
        assert sub * max(chunks) <= 256
        return sub
    return run


@pytest.mark.parametrize("sizes,sub", [
    ([1], 4), ([1 << 18], 4), ([(1 << 18) + 1], 2), ([1 << 19], 2), ([(1 << 19) + 1], 1),
    ([1 << 20], 1), ([(1 << 20) + 1], 0), ([100] * 20 + [(1 << 20) + 1], 0),
    ([16] * 5000, 4), ([16] * 100000, 0), ([2] * 8000, 0), ([64] * 8000, 2), ([64] * 30000, 0),
    ([256] * 30000, 2), ([16] * 6000 + [1 << 20], 1),
])
def test_rule(rule, sizes, sub):
    assert rule(sizes) == sub
