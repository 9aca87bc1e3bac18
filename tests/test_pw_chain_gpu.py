"""Consecutive pointwise layers in one launch (csrc/pw_chain.hip), by themselves and from a depthwise layer on: both tiles, whole and
odd frame counts, tiles without their second group, bias and relu, both forms of the rescale, activations of inner and last layers;
where a chain may not be formed."""
import numpy as np
import pytest

import oracle
import qasr_workloads as W
from qasr_workloads.nets import ACT_GLU, ACT_SIGMOID, ACT_SWISH, _Builder
from gpu_util import dev, GpuNet

pytestmark = pytest.mark.gpu


def check(net, launches, seed=3, s_for=None, **kw):
    """launches: {op name: (name of the op its launch begins with, kernel)}; kernel None: any but a chain's"""
    params = W.draw_net_params(net, seed, **kw)
    if s_for:
        for p in params:
            p["s"] = np.full_like(p["s"], s_for)
    x = W.draw_input(net, seed)
    ref = oracle.encoder_forward(net, params, x)
    g = GpuNet(net, params)
    names = [o.name for o in net.ops]
    for op, want in launches.items():
        first, kernel = g.enc.op_launch(names.index(op))
        assert names[first] == want[0] and (kernel == want[1] or (want[1] is None and kernel != "pw_chain")), (op, names[first], kernel)
    print(f"[case] chain {net.name} B={net.B} T={net.Tin}", flush=True)
    got = g.forward(dev(x)).cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} of {ref.size} differ, first at {bad[0]}"
    g.check_guards()
    g.y.zero_()
    g.enc.forward_layerwise(dev(x), g.y, g.ws)
    assert np.array_equal(g.y.cpu().numpy(), ref)
    g.enc.close()


def pointwise(B, T, widths, acts=(), relu=True, bias=True):
    b = _Builder("pointwise", 97, B, widths[0], T)
    for i, c in enumerate(widths[1:]):
        b.op(f"p{i}", c, relu=relu and i % 2 == 0, bias=bias or i % 2 == 1, act=acts[i] if i < len(acts) else 0)
    return b.done()


FORCE = "QASR_PW_CHAIN"


@pytest.mark.parametrize("MT", ["1", "2"])
@pytest.mark.parametrize("B,T", [(1, 16), (1, 17), (2, 31), (3, 48), (1, 213)])
@pytest.mark.parametrize("widths", [(512, 512, 512), (512, 2048, 512, 1024), (1024, 512, 1536, 512, 512), (2048, 512, 2048),
                                    (2048, 2048, 2048)])
def test_pointwise_chains(widths, B, T, MT, tuning_env):
    tuning_env(FORCE, "1")
    tuning_env("QASR_CHAIN_MT", MT)
    n = len(widths) - 1
    if MT == "2" and widths[1] == 2048 and widths[0] == 2048:     # two buffers of 2048 channels and the constants: one group only
        check(pointwise(B, T, widths), {"p0": ("p0", None), "p1": ("p1", None)})
    else:
        check(pointwise(B, T, widths, bias=T != 48), {f"p{n - 1}": ("p0", "pw_chain")})


@pytest.mark.parametrize("s", [20, 33, 62])
def test_limits_of_the_short_rescale(s, tuning_env):
    tuning_env(FORCE, "1")
    check(pointwise(1, 40, (512, 512, 512)), {"p1": ("p0", "pw_chain")}, s_for=s)


def conformer_tail(B, T, k, nonlinear):
    """From a depthwise layer on to a pointwise one whose GLU outputs the next reads as a prefix."""
    sw, glu = (ACT_SWISH, ACT_GLU) if nonlinear else (0, 0)
    b = _Builder("conformer_tail", 98, B, 512, T)
    b.op("in", 512, relu=False)
    b.op("dw", 512, k=k, groups=512, relu=False, bias=k % 2 == 1, act=sw)
    b.op("pw", 512, relu=False)
    b.op("up", 2048, act=sw)
    b.op("down", 512, relu=False)
    b.op("gate", 1024, relu=False, act=glu)
    b.op("half", 256, relu=False, Cin=512, x_batch_stride=1024 * b.T)
    return b.done()


@pytest.mark.parametrize("MT", ["1", "2"])
@pytest.mark.parametrize("B,T,k,nonlinear", [(1, 16, 32, True), (2, 33, 31, True), (1, 100, 42, False), (3, 61, 32, True), (2, 47, 3, True)])
def test_from_a_depthwise_layer_on(B, T, k, nonlinear, MT, tuning_env):
    tuning_env(FORCE, "1")
    tuning_env("QASR_CHAIN_MT", MT)
    check(conformer_tail(B, T, k, nonlinear), {"dw": ("dw", "pw_chain"), "gate": ("dw", "pw_chain")})


def test_longer_taps_keep_the_pair(tuning_env):
    tuning_env(FORCE, "1")
    check(conformer_tail(1, 64, 51, True), {"pw": ("dw", "sep"), "gate": ("up", "pw_chain")})


@pytest.mark.parametrize("glu_s", [30, 45])
def test_activations_of_a_chain(glu_s, tuning_env):
    tuning_env(FORCE, "1")
    b = _Builder("acts", 96, 2, 512, 50)
    b.op("a", 512, act=ACT_SIGMOID)
    b.op("b", 512, relu=False, act=ACT_SWISH)
    b.op("c", 1024, relu=False, act=ACT_GLU)
    b.op("d", 64, relu=False, Cin=512, x_batch_stride=1024 * b.T)
    net = b.done()
    params = W.draw_net_params(net, 2)
    for p in params:
        if p.get("act") and p["act"]["kind"] == ACT_SIGMOID:
            p["act"]["s"] = 39
        if p.get("act") and p["act"]["kind"] == ACT_GLU:
            p["act"]["s"] = glu_s
            p["act"]["m"] = p["act"]["m"] >> (45 - glu_s)
    x = W.draw_input(net, 2)
    g = GpuNet(net, params)
    assert [g.enc.op_launch(i) for i in range(3)] == [(0, "pw_chain")] * 3
    assert np.array_equal(g.forward(dev(x)).cpu().numpy(), oracle.encoder_forward(net, params, x))
    g.check_guards()
    g.enc.close()


def test_no_chain_through_what_others_read(tuning_env):
    """a second reader, a residual operand, all channels of a GLU's slot, a GLU as the network's output"""
    tuning_env(FORCE, "1")
    b = _Builder("second_reader", 95, 1, 512, 40)
    b.op("a", 512)
    m = b.op("b", 512)
    b.op("c", 512)
    b.op("d", 512, res=m)
    check(b.done(), {"a": ("a", "pw_chain"), "b": ("a", "pw_chain"), "c": ("c", None), "d": ("d", None)})
    b = _Builder("whole_slot", 94, 1, 512, 40)
    b.op("a", 512)
    b.op("b", 1024, relu=False, act=ACT_GLU)
    b.op("c", 512)
    check(b.done(), {"a": ("a", None), "b": ("b", None), "c": ("c", None)})
    b = _Builder("glu_out", 93, 1, 512, 40)
    b.op("a", 512)
    b.op("b", 1024, relu=False, act=ACT_GLU)
    check(b.done(), {"a": ("a", None), "b": ("b", None)})


def test_the_library_chooses_chains_for_a_conformer():
    """16 x 400 frames: from each depthwise layer to the next; the last pair by itself"""
    net = W.conformer_shaped(16, 400, 4, layers=2, nonlinear=True)
    check(net, {"L0.ffn1": ("L0.ffn1", "pw_chain"), "L0.pw1": ("L0.ffn1", "pw_chain"), "L0.dw": ("L0.dw", "pw_chain"),
                "L1.pw1": ("L0.dw", "pw_chain"), "L1.pw2": ("L1.dw", "sep")})
