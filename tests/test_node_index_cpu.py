"""Index arithmetic of the grid kernels (csrc/msm_index.hpp), compiled for the
host and compared with integer division for every node of grids up to the
2^28 nodes a plan accepts, and for every image of a node (no GPU needed)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1402_7216_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "msm_index.hpp"
// wrong nodes of a grid n0 x n1 x n2, or, with four numbers, wrong image
// ranges of the first and last nodes of periods around p with G ghosts
int main(int argc, char** argv) {
  const int n[3] = {atoi(argv[1]), atoi(argv[2]), atoi(argv[3])};
  long wrong = 0;
  if (argc == 4) {
    const int count = n[0] * n[1] * n[2];
    int node = 0;
    for (int z = 0; z < n[2]; ++z)
      for (int y = 0; y < n[1]; ++y)
        for (int x = 0; x < n[0]; ++x, ++node) {
          int m[3];
          msm::node_position(node, n, count, m);
          wrong += m[0] != x || m[1] != y || m[2] != z;
        }
  } else {
    for (int p = n[0]; p < n[0] + n[1]; ++p)
      for (int G = 1; G < n[2]; ++G)
        for (int k = 0; k < 2 * n[2]; ++k) {
          const int i = k < n[2] ? k % p : p - 1 - (k - n[2]) % p;
          const msm::ImageRange r = msm::image_range(i, p, G);
          const int below = (i + G) / p, above = (p + G - 1 - i) / p;
          wrong += r.first != -below || r.count != below + above + 1;
        }
  }
  std::printf("%ld\n", wrong);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("index")
    (d / "index.cpp").write_text(PROGRAM)
    exe = str(d / "index")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                    "-o", exe, str(d / "index.cpp")], check=True)
    return lambda *a: int(subprocess.run([exe, *map(str, a)], check=True, capture_output=True, text=True).stdout)


@pytest.mark.parametrize("n", [(1, 1, 1), (4, 5, 3), (161, 161, 161), (2048, 2048, 1), (2048, 2049, 1),
                               (182, 182, 182), (210, 210, 210), (422, 422, 422), (645, 645, 645), (4, 4, 16777216),
                               (16777216, 4, 4), (5, 53687091, 1)])
def test_node_positions_are_exact(program, n):
    assert program(*n) == 0


@pytest.mark.parametrize("period", [1, 2, 7, 160, 1 << 20, (1 << 22) - 20, 5400000])
def test_image_ranges_are_exact(program, period):
    assert program(period, 40, 17, 1) == 0
