"""The refinement's join of concurrent vertices (csrc/refine_join.hpp) over all
interleavings of its operations, on the CPU: join_interleavings.cpp runs the
code that the kernel runs, one operation on shared memory at a time."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def explorer(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("join") / "join_interleavings")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2405_11658_amd", "csrc"),
                    os.path.join(ROOT, "tests", "join_interleavings.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("tries,n,edges", [
    (3, 2, [(0, 1)]),                     # two that choose each other
    (2, 3, [(0, 1), (1, 2)]),             # one joins where another has just left
    (2, 3, [(1, 0), (0, 2)]),             # (weights of the three the other way round)
    (1, 3, [(0, 1), (1, 2), (0, 2)]),
    (1, 4, [(0, 1), (1, 2), (2, 3)]),
    (1, 4, [(0, 1), (0, 2), (0, 3)]),
])
def test_joins_leave_connected_communities(explorer, tries, n, edges):
    """Whatever the order: every community is connected and holds its
    representative, and its total is its members' weight exactly."""
    args = [str(x) for x in (tries, n, *sum(edges, ()))]
    r = subprocess.run([explorer] + args, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout
