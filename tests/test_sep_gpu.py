"""Depthwise + pointwise pairs that an encoder runs as one launch (csrc/sep.hip): every tile shape and
tap range, rows aligned and ragged, residual, both clamps of both layers, the 64-bit rescale, an
activation between the two layers, against the oracle; the same encoder layer by layer gives the
same bytes."""
import numpy as np
import pytest

import oracle
import qasr_workloads as W
from qasr_workloads.nets import _Builder
from gpu_util import dev, GpuNet

pytestmark = pytest.mark.gpu


def chain(B, T, C, Cout, k, dil=1, dw_relu=False, pw_relu=True, res=False, act=0, dw_bias=False):
    b = _Builder("sep_chain", 90, B, 64, T)
    b.op("in", C, k=3)
    r = b.op("proj", Cout, relu=False, advance=False) if res else -1
    b.op("dw", C, k=k, dilation=dil, groups=C, relu=dw_relu, bias=dw_bias, act=act)
    b.op("pw", Cout, relu=pw_relu, res=r)
    b.op("out", 29, relu=False)
    return b.done()


def check(net, seed=3, **kw):
    params = W.draw_net_params(net, seed, **kw)
    x = W.draw_input(net, seed)
    ref = oracle.encoder_forward(net, params, x)
    g = GpuNet(net, params)
    dw = [o.depthwise for o in net.ops].index(True)
    assert g.enc.op_launch(dw) == (dw, "sep") and g.enc.op_launch(dw + 1) == (dw, "sep")
    got = g.forward(dev(x)).cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} of {ref.size} differ, first at {bad[0]}"
    g.check_guards()
    g.y.zero_()
    g.enc.forward_layerwise(dev(x), g.y, g.ws)
    assert np.array_equal(g.y.cpu().numpy(), ref)
    g.y.zero_()
    ms = g.enc.forward_timed(dev(x), g.y, g.ws)      # a time per launch
    assert [i for i, t in enumerate(ms) if t == 0.0] == [dw + 1], ms
    assert np.array_equal(g.y.cpu().numpy(), ref)
    g.enc.close()


@pytest.mark.parametrize("tile", ["1,1", "2,1", "2,2", "4,1", "4,2", "7,1", "7,2"])
@pytest.mark.parametrize("C,Cout,k", [(256, 256, 33), (256, 512, 51), (512, 512, 63), (512, 512, 75), (512, 256, 39)])
def test_tile_shapes(C, Cout, k, tile, tuning_env):
    if Cout % (256 * int(tile[2])):
        pytest.skip("a workgroup takes 256 or 512 output channels")
    print(f"[case] sep {C}->{Cout} k={k} tile {tile}", flush=True)
    tuning_env("QASR_SEP", tile)
    check(chain(2, 272, C, Cout, k, res=k in (51, 75)))


@pytest.mark.parametrize("kw", [
    dict(B=1, T=16, C=256, Cout=256, k=1), dict(B=1, T=7, C=256, Cout=256, k=85), dict(B=3, T=113, C=512, Cout=512, k=32, res=True),
    dict(B=2, T=160, C=512, Cout=512, k=45, dil=2), dict(B=2, T=96, C=256, Cout=256, k=3, dw_relu=True, pw_relu=False, dw_bias=True),
    dict(B=5, T=230, C=256, Cout=512, k=13, act=2, pw_relu=False), dict(B=2, T=65, C=512, Cout=512, k=31, act=1, res=True, pw_relu=False)],
    ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()))
def test_options_and_edges(kw):
    print(f"[case] sep {kw}", flush=True)
    check(chain(**kw))


@pytest.mark.parametrize("lo,hi", [(20, 40), (33, 33), (54, 62)])
def test_rescale_ranges(lo, hi):
    """Shifts on either side of the short form's range, with a residual (which it adds before the shift)."""
    print(f"[case] sep s in {lo}..{hi}", flush=True)
    check(chain(2, 144, 256, 256, 33, res=True), s_lo=lo, s_hi=hi)


@pytest.mark.parametrize("T", [200, 203, 4])
def test_pair_is_the_whole_encoder(T):
    """Input and output are the caller's dense rows: loaded and stored at any byte address."""
    print(f"[case] separable module T={T}", flush=True)
    check(W.separable_module(3, 256, T, 33))


@pytest.mark.parametrize("T", [47, 48])
def test_padded_pointwise_layers_stay_apart(T):
    """Pointwise layers padded on the right: frames past their input are zeros to them."""
    b = _Builder("sep_padded", 96, 2, 64, T)
    b.op("in", 256, k=3)
    r = b.op("proj", 256, relu=False, pad=(0, 1), advance=False)
    b.op("dw", 256, k=33, groups=256, relu=False, bias=False, pad=(16, 17))
    b.op("pw", 256, res=r)
    b.op("dw2", 256, k=33, groups=256, relu=False, bias=False)
    b.op("pw2", 256, pad=(0, 1))
    b.op("out", 29, relu=False)
    net = b.done()
    params, x = W.draw_net_params(net, 6), W.draw_input(net, 6)
    g = GpuNet(net, params)
    print(f"[case] padded pointwise layers, T={T}", flush=True)
    assert [g.enc.op_launch(i)[0] for i in range(1, 6)] == [1, 2, 2, 4, 5]
    assert np.array_equal(g.forward(dev(x)).cpu().numpy(), oracle.encoder_forward(net, params, x))
    g.check_guards()
    g.enc.close()
