"""Host logic of the GNEB graphs (compiled with g++, no GPU): which captured
graphs a call makes, and what a capture that fails leaves.  A failed run of
eight iterations must leave the graph of one iteration in use and must not be
tried again; without the graph of one iteration nothing more is tried."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2605_26016_amd", "csrc")

# argv: fail0 fail1 n_iter...; per call: graphs tried, the two in hand, on, run_on
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "spx_gneb_graphs.hpp"
using namespace spx;
int main(int argc, char **argv) {
    const bool fail[2] = {std::atoi(argv[1]) != 0, std::atoi(argv[2]) != 0};
    GnebGraphs u;
    bool have[2] = {false, false};
    for (int k = 3; k < argc; ++k) {
        int tried = 0;
        make_gneb_graphs(u, have[0], have[1], std::atoi(argv[k]), [&](int q) {
            tried |= 1 << q;
            have[q] = !fail[q];
            return have[q];
        });
        std::printf("%d %d %d %d %d\n", tried, (int)have[0], (int)have[1], (int)u.on, (int)u.run_on);
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("graphs")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run([gxx, "-O1", "-std=c++17", "-Wall", "-I", CSRC, "-o", str(d / "p"), str(d / "p.cpp")], check=True)
    return str(d / "p")


@pytest.mark.parametrize("fail,calls,want", [
    ((0, 0), (1, 2, 120, 7, 8, 8), [(0, 0, 0, 1, 1), (1, 1, 0, 1, 1), (0, 1, 0, 1, 1), (0, 1, 0, 1, 1),
                                    (2, 1, 1, 1, 1), (0, 1, 1, 1, 1)]),
    ((0, 0), (200,), [(3, 1, 1, 1, 1)]),
    ((0, 1), (200, 200, 2), [(3, 1, 0, 1, 0), (0, 1, 0, 1, 0), (0, 1, 0, 1, 0)]),
    ((1, 0), (200, 200), [(1, 0, 0, 0, 1), (0, 0, 0, 0, 1)]),
], ids=["made_in_turn", "made_at_once", "run_fails", "one_fails"])
def test_graphs_made_and_kept(program, fail, calls, want):
    out = subprocess.run([program, *map(str, fail), *map(str, calls)], check=True, capture_output=True, text=True)
    assert [tuple(map(int, ln.split())) for ln in out.stdout.splitlines()] == want
