"""The node kernels' index maps (csrc/node_order.hpp), compiled for the host: division by the
box edge against the integer division, and the block order against a permutation."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_14505_amd", "csrc")

# The quotient is monotone in i, so it is right everywhere if it is right on both sides of
# every multiple of n below the box's n^3 nodes.
PROGRAM = r"""
#include "node_order.hpp"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace stgv;
int main(int, char** argv) {
  for (int n = atoi(argv[1]); n <= atoi(argv[2]); ++n) {
    const Geometry g = make_geometry(n, 0);
    for (uint32_t q = 0; q < (uint32_t)n * n; ++q)
      if (over_n(q * n, g) != q || over_n(q * n + n - 1, g) != q) { printf("n %d: quotient %u\n", n, q); return 1; }
    const uint32_t blocks = (g.n3 + node_threads(n) - 1) / node_threads(n);
    std::vector<char> seen(blocks, 0);
    for (uint32_t b = 0; b < blocks; ++b) {
      const uint32_t to = block_at(b, blocks, g);
      if (to >= blocks || seen[to]) { printf("n %d: block %u -> %u\n", n, b, to); return 1; }
      seen[to] = 1;
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("node_order")
    (d / "check.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, str(d / "check.cpp"), "-o", str(d / "check")], check=True)
    return str(d / "check")


@pytest.mark.parametrize("lo,hi", [(4, 64), (65, 200), (250, 260), (384, 385), (511, 513), (1023, 1024)])
def test_division_and_block_order(program, lo, hi):
    r = subprocess.run([program, str(lo), str(hi)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


SMALL_STATES = r"""
#include "node_order.hpp"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace stgv;
int main() {
  for (int n = 4; n <= 96; ++n) {
    const Geometry g = make_geometry(n, 0, true);
    const uint32_t blocks = (g.n3 + node_threads(n) - 1) / node_threads(n);
    std::vector<char> seen(blocks, 0);
    uint32_t last[8] = {};
    for (uint32_t b = 0; b < blocks; ++b) {
      const uint32_t even = block_at(b, blocks, g, false), odd = block_at(b, blocks, g, true);
      if (even != odd) { printf("n %d: workgroup %u holds block %u in even steps, %u in odd ones\n", n, b, even, odd); return 1; }
      if (even >= blocks || seen[even]) { printf("n %d: block %u -> %u\n", n, b, even); return 1; }
      seen[even] = 1;
      if (b >= 8 && even != last[b % 8] + 1) { printf("n %d: XCD %u has a gap at %u\n", n, b % 8, even); return 1; }
      last[b % 8] = even;
    }
    // what a state beyond the L2s takes is untouched
    const Geometry far = make_geometry(n, 0);
    if (far.slab || block_at(0, blocks, far, false) != 0 || block_at(blocks - 1, blocks, far, false) != blocks - 1) return 1;
  }
  return 0;
}
"""


def test_small_states_keep_a_node_on_one_xcd(tmp_path):
    # every step of a small state gives a block to the same XCD, in one run of consecutive blocks
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    (tmp_path / "check.cpp").write_text(SMALL_STATES)
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, str(tmp_path / "check.cpp"), "-o", str(tmp_path / "check")], check=True)
    r = subprocess.run([str(tmp_path / "check")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
