"""Consecutive pointwise layers in one launch (csrc/pw_chain.hip), by themselves and from a depthwise layer on: both tiles, whole and
odd frame counts, tiles without their second group, bias and relu, both forms of the rescale, activations of inner and last layers;
where a chain may not be formed."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("MT", ["1", "2", "4"])
@pytest.mark.parametrize("k", [45, 53, 69, 87])
def test_a_pairs_table_beside_its_rows(k, MT, tuning_env):
    """Every range of taps: rows in LDS end where the activation's table begins."""
    tuning_env(FORCE, "1")
    tuning_env("QASR_SEP", MT)
    for T in (16, 64, 213):
        check(conformer_tail(1, T, k, True), {"pw": ("dw", "sep")})


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


def test_activations_in_separate_launches(tuning_env):
    """The Conformer whose layers the library runs as chains, without them: Swish in the layers' epilogues, GLU in place."""
    tuning_env("QASR_NO_PW_CHAIN", "1")
    net = W.conformer_shaped(16, 400, 4, layers=2, nonlinear=True)
    check(net, {o.name: (o.name if not o.name.endswith("pw2") else o.name[:-3] + "dw", None) for o in net.ops})


def test_chains_apply_what_layers_by_themselves_do_apart():
    net = W.conformer_shaped(16, 400, 4, layers=2, nonlinear=True)
    g = GpuNet(net, W.draw_net_params(net, 1))
    seen = {(o.act, g.enc.op_launch(i)[1], g.enc.op_act_fused(i)) for i, o in enumerate(net.ops) if o.act}
    assert seen >= {(ACT_GLU, "pw_chain", False), (ACT_SWISH, "pw_chain", True)}
    g.enc.close()


@pytest.mark.parametrize("s", [20, 33, 62])
@pytest.mark.parametrize("relu", [True, False])
def test_relu_and_rescales_of_the_depthwise_layer(s, relu, tuning_env):
    """Its epilogue's three forms; the other layers keep theirs."""
    tuning_env(FORCE, "1")
    net = conformer_tail(2, 45, 31, False)
    net.ops[1].flags = 1 if relu else 0
    params = W.draw_net_params(net, 4)
    params[1]["s"] = np.full_like(params[1]["s"], s)
    if s == 20:
        params[1]["m"] = params[1]["m"] >> 18            # (codes over the whole range, not two)
    x = W.draw_input(net, 4)
    ref, outs = oracle.encoder_forward(net, params, x, keep=True)
    assert s == 62 or len(np.unique(outs[1])) > 16
    g = GpuNet(net, params)
    assert g.enc.op_launch(1) == (1, "pw_chain")
    assert np.array_equal(g.forward(dev(x)).cpu().numpy(), ref)
    g.check_guards()
    g.enc.close()


@pytest.mark.parametrize("B,T", [(1, 16 * 300), (3, 16 * 100 - 5)])
def test_more_tiles_than_units(B, T, tuning_env):
    """A second round of workgroups, which only a forced chain has."""
    tuning_env(FORCE, "1")
    tuning_env("QASR_CHAIN_MT", "1")
    check(pointwise(B, T, (512, 512, 512)), {"p1": ("p0", "pw_chain")})


def to_the_output(B, T, k=31):
    b = _Builder("to_the_output", 91, B, 512, T)
    b.op("in", 512, relu=False)
    b.op("dw", 512, k=k, groups=512, relu=False)
    b.op("pw", 512)
    b.op("up", 1024, relu=False)
    return b.done()


@pytest.mark.parametrize("MT", ["1", "2"])
@pytest.mark.parametrize("B,T", [(1, 61), (2, 100), (3, 16), (2, 33)])
def test_from_a_depthwise_layer_to_the_output(B, T, MT, tuning_env):
    tuning_env(FORCE, "1")
    tuning_env("QASR_CHAIN_MT", MT)
    check(to_the_output(B, T), {"dw": ("dw", "pw_chain"), "up": ("dw", "pw_chain")})


@pytest.mark.parametrize("net", [lambda: pointwise(2, 48, (512, 1024, 512)), lambda: pointwise(2, 37, (512, 1024, 512)),
                                 lambda: to_the_output(2, 48), lambda: to_the_output(2, 61)])
@pytest.mark.parametrize("dx,dy", [(1, 0), (0, 1), (3, 5), (16, 4)])
def test_input_and_output_at_any_address(net, dx, dy, tuning_env):
    tuning_env(FORCE, "1")
    net = net()
    params = W.draw_net_params(net, 8)
    x = W.draw_input(net, 8)
    ref = oracle.encoder_forward(net, params, x)
    g = GpuNet(net, params)
    xr = torch.full((x.size + dx,), 9, dtype=torch.int8, device="cuda")
    yr = torch.full((ref.size + dy + 64,), 9, dtype=torch.int8, device="cuda")
    xr[dx:] = dev(x).reshape(-1)
    y = yr[dy:dy + ref.size]
    g.enc.forward(xr[dx:], y, g.ws)
    assert np.array_equal(y.cpu().numpy().reshape(ref.shape), ref)
    assert bool((yr[:dy] == 9).all()) and bool((yr[dy + ref.size:] == 9).all())
    g.check_guards()
    g.enc.close()


@pytest.mark.parametrize("nonlinear", [False, True])
@pytest.mark.parametrize("B,T", [(2, 45), (2, 48)])
def test_other_entry_points(B, T, nonlinear, tuning_env):
    """Float features (rows of the network's ends rounded up to 16 frames), the library's own workspace, a graph replayed between
    eager forwards."""
    tuning_env(FORCE, "1")
    b = _Builder("entries", 90, B, 512, T)
    sw, glu = (ACT_SWISH, ACT_GLU) if nonlinear else (0, 0)
    for i in range(2):
        b.op(f"dw{i}", 512, k=32 - i, groups=512, relu=False, act=sw)
        b.op(f"pw{i}", 512, relu=False)
        b.op(f"up{i}", 1024, act=sw)
        b.op(f"gate{i}", 1024, relu=False, act=glu)
        b.op(f"half{i}", 256, relu=False, Cin=512, x_batch_stride=1024 * T)
        b.op(f"back{i}", 512, relu=False)
    net = b.done()
    params = W.draw_net_params(net, 7)
    xf = np.random.default_rng(7).normal(0, 2, (B, 512, T)).astype(np.float32)
    x = oracle.quantize(xf, 4.0)
    ref = oracle.encoder_forward(net, params, x)
    g = GpuNet(net, params)
    names = [g.enc.op_launch(i) for i in range(g.enc.n_ops)]
    assert names[7] == (6, "pw_chain") and (T % 16 or names[1] == (0, "pw_chain"))
    ws = torch.full((g.enc.workspace_bytes_f32,), 77, dtype=torch.int8, device="cuda")
    y = torch.empty(ref.shape, dtype=torch.float32, device="cuda")
    g.enc.forward_f32(dev(xf), 4.0, 0.25, y, ws)
    assert np.array_equal(y.cpu().numpy(), ref.astype(np.float32) * np.float32(0.25))
    xd = dev(x)
    g.enc.forward_static(xd, g.y)
    assert np.array_equal(g.y.cpu().numpy(), ref)
    graph = g.enc.graph(xd, g.y, g.ws)
    for i in range(3):
        other = W.draw_input(net, 20 + i)
        xd.copy_(torch.from_numpy(other))
        want = g.enc.forward_layerwise(xd, torch.empty_like(g.y), g.ws).cpu().numpy()
        g.ws.fill_(77)
        g.y.zero_()
        graph.launch()
        assert np.array_equal(g.y.cpu().numpy(), want)
    xd.copy_(torch.from_numpy(x))
    graph.launch()
    assert np.array_equal(g.y.cpu().numpy(), ref)
    graph.close()
    g.check_guards()
    g.enc.close()


def slots(net, *wires):
    for o, (i, j) in zip(net.ops, wires):
        o.in_slot, o.out_slot = i, j
    net.n_slots = 1 + max(max(w) for w in wires)
    return net


def test_a_chain_does_not_write_what_it_reads(tuning_env):
    """Where its last output would lie over its first input, a chain is shorter, or does not begin with its depthwise layer."""
    tuning_env(FORCE, "1")
    tuning_env("QASR_SLOT_DEPTH", "0")                # (slots are buffers)
    b = _Builder("over_itself", 89, 2, 512, 75)
    for n in ("in", "a", "b", "c", "d"):
        b.op(n, 512, relu=n == "b")
    b.op("end", 64, relu=False)
    wires = ((0, 1), (1, 2), (2, 1), (1, 2), (2, 1), (1, 3))
    # (from `in` on: four layers to slot 2; then d alone)
    check(slots(b.done(), *wires), {"in": ("in", "pw_chain"), "c": ("in", "pw_chain"), "d": ("d", None)})
    b = _Builder("over_itself_later", 88, 2, 512, 75)
    b.op("first", 512, k=3)
    for n in ("a", "b", "c", "d"):
        b.op(n, 512, relu=n == "b")
    b.op("end", 64, relu=False)
    # (a to d would read and write slot 1)
    check(slots(b.done(), *wires), {"a": ("a", "pw_chain"), "c": ("a", "pw_chain"), "d": ("d", None)})
    b = _Builder("over_its_depthwise_input", 87, 2, 512, 75)
    b.op("in", 512, relu=False)
    b.op("dw", 512, k=31, groups=512, relu=False)
    b.op("pw", 512)
    b.op("up", 1024)
    b.op("down", 512, relu=False)
    b.op("end", 64, relu=False)
    net = b.done()
    # (dw to down would read and write slot 1, whose neighbouring frames other workgroups read)
    check(slots(net, (0, 1), (1, 2), (2, 3), (3, 2), (2, 1), (1, 4)), {"dw": ("dw", "sep"), "pw": ("dw", "sep"), "up": ("up", "pw_chain"), "down": ("up", "pw_chain")})
    # (... and with a slot of its own it is one launch)
    check(slots(net, (0, 1), (1, 2), (2, 3), (3, 2), (2, 4), (4, 1)), {"dw": ("dw", "pw_chain"), "down": ("dw", "pw_chain")})


@pytest.mark.parametrize("depth", ["0", "1", "2"])
@pytest.mark.parametrize("nonlinear", [False, True])
def test_fewer_buffers(depth, nonlinear, tuning_env):
    tuning_env(FORCE, "1")
    tuning_env("QASR_SLOT_DEPTH", depth)
    net = W.conformer_shaped(2, 75, 4, layers=3, nonlinear=nonlinear)
    check(net, {"L0.ffn1": ("L0.ffn1", "pw_chain")})
