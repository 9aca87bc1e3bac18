"""Grid sizes of launches with one workgroup per unit of work, up to the most rows the integer softmax takes:
every dimension below 2^32 work items, every unit covered once (compiled for the host)."""
import os
import subprocess

import paper_2103_16827_amd as Q
from paper_2103_16827_amd.binding import make_desc

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2103_16827_amd", "csrc")

MAIN = r"""
#include "launch_shape.hpp"
#include <cstdio>
#include <initializer_list>
int main() {
  const int64_t units[] = {1, 2, 1000, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, (1ll << 30) - 1, 1ll << 30};
  for (int64_t n : units) {
    const qasr::GridShape g = qasr::grid_shape(n);
    const unsigned long long items = 1024ull * g.x;
    // the last workgroup of the last row, and of the row before, in the kernel's numbering
    const int64_t last = ((int64_t)(g.y - 1) << qasr::kGridShift) + g.x - 1;
    const bool whole = g.y == 1 || g.x == 1u << qasr::kGridShift;
    if (items >= 1ull << 32 || g.y > 65535 || !whole || last < n - 1 || last - g.x >= n - 1) {
      std::printf("%lld units: %u x %u\n", (long long)n, g.x, g.y);
      return 1;
    }
  }
  for (int threads : {256, 512, 1024})
    if (qasr::max_workgroups(threads) * threads >= 1ll << 32 || (qasr::max_workgroups(threads) + 8) * threads < 1ll << 32) return 2;
  return 0;
}
"""


def test_every_dimension_of_a_large_launch_is_accepted(tmp_path):
    src, exe = tmp_path / "shape.cpp", tmp_path / "shape"
    src.write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_long_pointwise_layers_leave_the_kernel_of_1024_threads():
    """64 -> 16 channels over 2^30 frames: more than 2^22 workgroups of pw_wide's largest tile."""
    assert Q.conv1d_launch_name(make_desc(64, 64, 16, 1 << 20, flags=Q.FLAG_W_PACKED)) == "pw_wide"
    assert Q.conv1d_launch_name(make_desc(1024, 64, 16, 1 << 20, flags=Q.FLAG_W_PACKED)) == "gemm_mfma"
