"""A residual projection (pointwise layer of a block's input) that runs in the launch of the pair after it
(csrc/sep.hip): every tile, odd frame counts, batches that leave the last round short, options of the projection;
the pair's own residual; not where the pair reads the projection."""
import numpy as np
import pytest

import oracle
import qasr_workloads as W
from qasr_workloads.nets import _Builder
from gpu_util import dev, GpuNet

pytestmark = pytest.mark.gpu


def block(B, T, C, Cout, k, proj_relu=False, proj_bias=True, pw_res=False):
    b = _Builder("proj_block", 91, B, 64, T)
    b.op("in", C, k=3)
    skip = -1
    if pw_res:
        skip = b.op("in2", Cout, relu=False, advance=False)
    r = b.op("proj", Cout, relu=proj_relu, bias=proj_bias, advance=False)
    b.op("dw1", C, k=k, groups=C, relu=False, bias=False)
    b.op("pw1", Cout, res=skip)
    b.op("dw2", Cout, k=33, groups=Cout, relu=False, bias=False)
    b.op("pw2", Cout, res=r)
    b.op("out", 29, relu=False)
    return b.done()


def check(net, fused=True, seed=5, **kw):
    params = W.draw_net_params(net, seed, **kw)
    x = W.draw_input(net, seed)
    ref = oracle.encoder_forward(net, params, x)
    g = GpuNet(net, params)
    i = [o.name for o in net.ops].index("proj")
    launches = [g.enc.op_launch(j) for j in (i, i + 1, i + 2)]
    assert (launches == [(i, "sep")] * 3) == fused, launches
    got = g.forward(dev(x)).cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} of {ref.size} differ, first at {bad[0]}"
    g.check_guards()
    g.y.zero_()
    g.enc.forward_layerwise(dev(x), g.y, g.ws)
    assert np.array_equal(g.y.cpu().numpy(), ref)
    if fused:
        ms = g.enc.forward_timed(dev(x), g.y, g.ws)
        assert ms[i] > 0 and ms[i + 1] == 0 and ms[i + 2] == 0
    g.enc.close()


TILES = ["", "1,1", "1,1,2", "2,1,2", "2,1", "2,2", "4,1", "4,2", "7,1", "7,2"]
SHAPES = [(256, 256, 33, 130), (256, 512, 51, 64), (512, 512, 75, 227), (512, 256, 63, 17)]


# (tiles of two columns per wave: a workgroup takes 512 output channels)
@pytest.mark.parametrize("C,Cout,k,T,tile", [s + (t,) for s in SHAPES for t in TILES if t not in ("2,2", "4,2", "7,2") or s[1] % 512 == 0])
def test_tiles(C, Cout, k, T, tile, tuning_env):
    print(f"[case] projection {C}->{Cout} k={k} T={T} tile {tile}", flush=True)
    if tile:
        tuning_env("QASR_SEP", tile)
    check(block(2, T, C, Cout, k))


@pytest.mark.parametrize("kw", [dict(proj_relu=True), dict(proj_bias=False), dict(pw_res=True)], ids=str)
def test_options(kw):
    print(f"[case] projection {kw}", flush=True)
    check(block(3, 70, 256, 256, 33, **kw))


def test_rescale_ranges():
    print("[case] projection s in 20..62", flush=True)
    check(block(1, 48, 256, 256, 33), s_lo=20, s_hi=62)


def test_other_tensors_stay_apart():
    """The projection of another tensor than the pair's input keeps a launch of its own."""
    b = _Builder("proj_other", 92, 2, 64, 80)
    a = b.op("in", 256, k=3)
    b.op("mid", 256)
    r = b.op("proj", 256, relu=False, advance=False, src=(a, 256))
    b.op("dw1", 256, k=33, groups=256, relu=False, bias=False)
    b.op("pw1", 256, res=r)
    b.op("out", 29, relu=False)
    print("[case] projection of another tensor", flush=True)
    check(b.done(), fused=False)
