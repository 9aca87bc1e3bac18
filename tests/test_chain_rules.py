"""Which runs of pointwise layers go out as one launch (csrc/pw_chain.hip), on either side of the rule's lines: the library's own
rule, asked by a small host program (no GPU)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(HERE, "..", "paper_2103_16827_amd")
CLANG = "/opt/rocm/llvm/bin/clang++"

MAIN = r"""
#include "kernels.hpp"
#include "pw_chain.hpp"
#include <cstdio>
#include <vector>
using qasr::ChainOp;
using qasr::ConvParams;
namespace {
ConvParams layer(int B, int Cin, int Cout, int T, int k, bool dense) {
  ConvParams p{};
  p.B = B; p.Cin = Cin; p.Cout = Cout; p.Tin = p.Tout = T;
  p.k = k; p.stride = p.dil = 1; p.pl = (k - 1) / 2; p.depthwise = k > 1; p.w_packed = k == 1;
  p.xpad = p.ypad = dense ? 0 : (16 - T % 16) % 16;           // (rows rounded up to 16 frames, as inside an encoder)
  p.xbs = (int64_t)Cin * (T + p.xpad); p.ybs = (int64_t)Cout * (T + p.ypad);
  return p;
}
int failed = 0;
void expect(bool want, const char* what, int B, int T, std::vector<int> widths, bool dw = false, bool glu = false, bool dense = false) {
  ChainOp op[qasr::kMaxChain]{};
  const int n = (int)widths.size() - 1;
  for (int i = 0; i < n; ++i) {
    op[i].p = layer(B, widths[i], widths[i + 1], T, 1, dense);
    op[i].glu = glu && i + 1 == n;
  }
  const ConvParams d = layer(B, 512, 512, T, 31, dense);
  const bool got = qasr::pw_chain_better(dw ? &d : nullptr, op, n);
  if (got != want) { std::printf("%s, %d x %d frames: %d\n", what, B, T, got); ++failed; }
}
}  // namespace
int main() {
  // whose rows out are wide: where the chain is not the faster way
  expect(false, "512 -> 512 -> 1024", 4, 800, {512, 512, 1024});
  expect(false, "512 -> 512 -> 1024", 10, 400, {512, 512, 1024});
  expect(true, "512 -> 512 -> 1024", 12, 400, {512, 512, 1024});
  expect(false, "512 -> 512 -> 2048", 16, 512, {512, 512, 2048});
  expect(true, "512 -> 512 -> 512 -> 1024", 16, 400, {512, 512, 512, 1024});
  expect(true, "512 -> 512 -> 1024 over odd rows", 4, 799, {512, 512, 1024}, false, false, true);
  expect(false, "512 -> 512 -> 512 -> 1024 over odd rows", 1, 104, {512, 512, 512, 1024}, false, false, true);
  expect(false, "512 -> 512 -> 1024 over odd frames in whole rows", 4, 799, {512, 512, 1024});
  // ... whose rows in are, of two groups
  expect(false, "2048 -> 512 -> 512", 16, 512, {2048, 512, 512});
  expect(true, "1024 -> 512 -> 512", 16, 400, {1024, 512, 512});
  // one round of workgroups: 256 tiles
  expect(true, "four layers", 16, 400, {512, 512, 512, 512, 512});
  expect(true, "four layers", 1, 16 * 512, {512, 512, 512, 512, 512});
  expect(false, "four layers", 1, 16 * 513, {512, 512, 512, 512, 512});
  expect(false, "four layers", 32, 400, {512, 512, 512, 512, 512});
  for (bool glu : {false, true}) {
    expect(true, "a Conformer's layer", 8, 400, {512, 512, 2048, 512, 1024}, true, glu);
    expect(true, "a Conformer's layer", 16, 400, {512, 512, 2048, 512, 1024}, true, glu);
    expect(false, "a Conformer's layer", 20, 400, {512, 512, 2048, 512, 1024}, true, glu);
    expect(false, "a Conformer's layer", 1, 400, {512, 512, 2048, 512, 1024}, true, glu);
  }
  expect(true, "two layers", 2, 400, {512, 512, 512});
  expect(false, "wide layers", 1, 400, {512, 2048, 512});
  return failed != 0;
}
"""


@pytest.mark.skipif(not os.path.exists(CLANG), reason="no host clang beside the HIP toolchain")
def test_chains_where_they_are_the_faster_way(tmp_path):
    src, exe = tmp_path / "chains.hip", tmp_path / "chains"
    src.write_text(MAIN)
    subprocess.check_call([CLANG, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-I", os.path.join(PKG, "csrc"), str(src),
                           "-x", "none", os.path.join(PKG, "libqasr.so"), f"-Wl,-rpath,{PKG}", "-L/opt/rocm/lib", "-lamdhip64",
                           "-Wl,-rpath,/opt/rocm/lib", "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
