"""CPU tests of the walk's stack of pending cells: its own source over 64 emulated lanes
(walk_stack_host.cpp)."""

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1106_1900_amd", "csrc")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("stack") / "walk_stack_host")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-w", "-I", CSRC,
                           os.path.join(HERE, "walk_stack_host.cpp"), "-o", exe])

    def run(*args):
        p = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60)
        assert p.returncode == 0, p.stdout
        return [int(x) for x in p.stdout.split()[1:]]
    return run


def test_nodes_without_children_push_nothing(host):
    # such a record is only met in an inconsistent tree, whose error is reported after the
    # walk; the walk has to end and stay in its memory all the same
    host("childless")


@pytest.mark.parametrize("children,levels", [(1, 60), (2, 12), (5, 6), (8, 5)])
def test_every_cell_is_popped_once(host, children, levels):
    host("tree", children, levels)


@pytest.mark.parametrize("children,levels", [(3, 9), (5, 7), (8, 6)])
def test_pops_keep_their_width(host, children, levels):
    # more cells pending than the LDS part holds, all of them opened
    most, spilled, narrowest = host("tree", children, levels)
    assert most > 384 and spilled > 0
    assert narrowest == 64


def test_stack_never_fills(host):
    # 20 levels of nodes with eight children each: the words in device memory run out, and
    # pops narrow instead
    most, spilled, narrowest = host("deep", 20)
    assert most > 5000 and 800 < spilled <= 1280
    assert narrowest < 64
