"""Several pointwise layers of equal output shape in one launch (csrc/pw_wide.hip): every tile, different input
widths, clamps and biases side by side, odd frame counts; a dense-residual stack; not where one layer reads
another's output."""
import numpy as np
import pytest

import oracle
import qasr_workloads as W
from qasr_workloads.nets import _Builder
from gpu_util import dev, GpuNet

pytestmark = pytest.mark.gpu


def block(B, T, widths, Cout, chained=False):
    b = _Builder("multi_block", 92, B, 64, T)
    src = []
    for i, C in enumerate(widths):
        b.op(f"in{i}", C, k=3)
        src.append((b.cur, C))
    more = []
    for i, s in enumerate(src):
        if chained and i == 1:
            s = (more[0], Cout)
        more.append(b.op(f"proj{i}", Cout, relu=i % 2 == 1, bias=i != 2, advance=False, src=s))
    b.op("conv", Cout, k=5, res=more[0], more_res=more[1:])
    b.op("out", 29, relu=False)
    return b.done()


def check(net, n, fused=True, seed=7, **kw):
    params = W.draw_net_params(net, seed, **kw)
    x = W.draw_input(net, seed)
    ref = oracle.encoder_forward(net, params, x)
    g = GpuNet(net, params)
    i = [o.name for o in net.ops].index("proj0")
    launches = [g.enc.op_launch(j)[0] for j in range(i, i + n)]
    assert (launches == [i] * n) == fused, launches
    got = g.forward(dev(x)).cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} of {ref.size} differ, first at {bad[0]}"
    g.check_guards()
    g.y.zero_()
    g.enc.forward_layerwise(dev(x), g.y, g.ws)
    assert np.array_equal(g.y.cpu().numpy(), ref)
    if fused:
        ms = g.enc.forward_timed(dev(x), g.y, g.ws)
        assert ms[i] > 0 and all(ms[j] == 0 for j in range(i + 1, i + n))
    g.enc.close()


@pytest.mark.parametrize("tile", ["", "1,1", "2,1", "4,1", "7,1", "1,2", "2,2", "4,2", "7,2", "1,4", "2,4", "4,4", "1,8", "2,8", "4,8"])
@pytest.mark.parametrize("widths,Cout,B,T", [((512, 512), 512, 2, 60), ((512, 768, 640), 1024, 1, 129),
                                             ((512, 576, 512, 832, 512), 200, 3, 31)])
def test_tiles(widths, Cout, B, T, tile, tuning_env):
    print(f"[case] {widths} -> {Cout}, B={B} T={T}, tile {tile}", flush=True)
    if tile:
        tuning_env("QASR_PWW", tile)
    check(block(B, T, widths, Cout), len(widths))


def test_input_of_few_channels():
    """no more groups over the input channels than the narrowest layer has chunks"""
    check(block(1, 40, (64, 768), 256), 2)


def test_layer_that_reads_another_runs_after_it():
    check(block(1, 70, (512, 512, 512), 512, chained=True), 3, fused=False)


def test_dense_residual_stack():
    """ten projections and more, every block's from the inputs of all blocks before it"""
    b = _Builder("multi_dense", 93, 1, 64, 90)
    b.op("pro", 256, k=3)
    src = []
    for blk in range(12):
        src.append((b.cur, b.C))
        more = [b.op(f"{blk}.res{j}", 256, relu=False, advance=False, src=s) for j, s in enumerate(src)]
        b.op(f"{blk}.conv", 256, k=3, res=more[0], more_res=more[1:])
    b.op("out", 29, relu=False)
    net = b.done()
    params = W.draw_net_params(net, 3)
    x = W.draw_input(net, 3)
    g = GpuNet(net, params)
    names = [o.name for o in net.ops]
    for blk in range(1, 12):
        i = names.index(f"{blk}.res0")
        assert {g.enc.op_launch(j) for j in range(i, i + blk + 1)} == {(i, "pw_wide")}
    assert np.array_equal(g.forward(dev(x)).cpu().numpy(), oracle.encoder_forward(net, params, x))
    g.check_guards()
    g.enc.close()


def test_second_half_of_a_pair_stays_with_it():
    """a pointwise layer that runs with the depthwise layer before it does not begin a launch of several"""
    b = _Builder("multi_pair", 95, 1, 64, 90)
    b.op("in", 256, k=3)
    src = (b.cur, b.C)
    b.op("dw", 256, k=33, groups=256, relu=False, bias=False)
    b.op("pw", 256)
    r = b.op("proj", 256, relu=False, advance=False, src=src)
    b.op("conv", 256, k=3, res=r)
    b.op("out", 29, relu=False)
    net = b.done()
    params = W.draw_net_params(net, 8)
    x = W.draw_input(net, 8)
    g = GpuNet(net, params)
    i = [o.name for o in net.ops].index("dw")
    assert [g.enc.op_launch(j)[0] for j in (i, i + 1, i + 2)] == [i, i, i + 2]
    ms = g.enc.forward_timed(dev(x), g.y, g.ws)
    assert ms[i] > 0 and ms[i + 1] == 0 and ms[i + 2] > 0
    assert np.array_equal(g.forward(dev(x)).cpu().numpy(), oracle.encoder_forward(net, params, x))
    g.check_guards()
    g.enc.close()
