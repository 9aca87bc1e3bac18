"""Which layers may run as a depthwise + pointwise pair, and take a projection along (csrc/sep.hip), by their geometry, and
with which tile: the library's own rules, asked by a small host program (no GPU)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(HERE, "..", "paper_2103_16827_amd")
CLANG = "/opt/rocm/llvm/bin/clang++"

MAIN = r"""
#include "kernels.hpp"
#include "sep.hpp"
#include <cstdio>
using qasr::ConvParams;
namespace {
// rows rounded up to 16 frames, as inside an encoder
ConvParams layer(int B, int Cin, int Cout, int T, int k, int pl, int pr, int dw) {
  ConvParams p{};
  p.B = B; p.Cin = Cin; p.Cout = Cout; p.Tin = T; p.Tout = T + pl + pr - (k - 1);
  p.k = k; p.stride = p.dil = 1; p.pl = pl; p.depthwise = dw; p.w_packed = !dw;
  p.xpad = (16 - p.Tin % 16) % 16; p.ypad = (16 - p.Tout % 16) % 16;
  p.xbs = (int64_t)Cin * (p.Tin + p.xpad); p.ybs = (int64_t)Cout * (p.Tout + p.ypad);
  return p;
}
int failed = 0;
void expect(const char* what, int T, bool got, bool want) {
  if (got != want) { std::printf("%s, %d frames: %d\n", what, T, got); ++failed; }
}
}  // namespace
int main() {
  for (int T : {48, 793, 799, 800}) {
    const ConvParams d = layer(2, 256, 256, T, 33, 16, 16, 1), q = layer(2, 256, 256, T, 1, 0, 0, 0), r = q;
    expect("pair", T, qasr::sep_supported(d, q), true);
    expect("projection", T, qasr::sep_projection_supported(d, q, r), true);
    // a pointwise layer padded on the right has frames past its input, where it sees zeros and not what the
    // depthwise layer, or the bytes between rows, would have there
    expect("padded pair", T, qasr::sep_supported(d, layer(2, 256, 256, T, 1, 0, 1, 0)), false);
    expect("padded projection", T, qasr::sep_projection_supported(d, q, layer(2, 256, 256, T, 1, 0, 1, 0)), false);
    const ConvParams dl = layer(2, 256, 256, T, 33, 16, 17, 1), ql = layer(2, 256, 256, T + 1, 1, 0, 0, 0);
    expect("longer pair", T, qasr::sep_supported(dl, ql), true);
    expect("padded projection of a longer pair", T, qasr::sep_projection_supported(dl, ql, layer(2, 256, 256, T, 1, 0, 1, 0)), false);
  }
  // tiles (groups of 16 frames, 16-channel columns per wave), where another takes 1.2 to 1.35 of their time
  struct { int C, k, B, T; bool projection; int MT, NT; } tiles[] = {
    {512, 45, 45, 1265, false, 4, 2}, {512, 45, 36, 1720, false, 4, 2},
    {512, 75, 2, 368, true, 1, 1}, {512, 81, 3, 697, true, 2, 1}, {512, 45, 6, 352, true, 2, 1}, {512, 57, 9, 304, true, 2, 2},
    {512, 69, 39, 70, true, 2, 2}, {512, 51, 8, 800, true, 4, 2}, {512, 63, 7, 832, true, 4, 2}, {256, 87, 3, 960, true, 2, 1},
  };
  for (const auto& t : tiles) {
    const ConvParams d = layer(t.B, t.C, t.C, t.T, t.k, (t.k - 1) / 2, (t.k - 1) / 2, 1), q = layer(t.B, t.C, t.C, t.T, 1, 0, 0, 0);
    qasr::SepChoice c{};
    if (!qasr::sep_choice(d, q, t.projection, c) || c.MT != t.MT || c.NT != t.NT) {
      std::printf("%d channels, %d taps, %d x %d frames: tile %d x %d\n", t.C, t.k, t.B, t.T, c.MT, c.NT);
      ++failed;
    }
  }
  return failed != 0;
}
"""


@pytest.mark.skipif(not os.path.exists(CLANG), reason="no host clang beside the HIP toolchain")
def test_padded_pointwise_layers_keep_launches_of_their_own_and_tiles_are_the_fastest(tmp_path):
    src, exe = tmp_path / "pairs.hip", tmp_path / "pairs"
    src.write_text(MAIN)
    subprocess.check_call([CLANG, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-I", os.path.join(PKG, "csrc"), str(src),
                           "-x", "none", os.path.join(PKG, "libqasr.so"), f"-Wl,-rpath,{PKG}", "-L/opt/rocm/lib", "-lamdhip64",
                           "-Wl,-rpath,/opt/rocm/lib", "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
