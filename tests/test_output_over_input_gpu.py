"""Forwards whose output lies over their input: the last layer writes where the first one read, so the two never share a launch."""
import numpy as np
import pytest
import torch

import oracle
import qasr_workloads as W
from qasr_workloads.nets import _Builder
from gpu_util import FILL, GpuNet, dev

pytestmark = pytest.mark.gpu


def pair(B, T):
    b = _Builder("pair", 92, B, 256, T)
    b.op("dw", 256, k=33, groups=256, relu=False)
    b.op("pw", 256)
    return b.done(), False


def chain(B, T):
    b = _Builder("chain", 92, B, 512, T)
    b.op("a", 1024)
    b.op("b", 512, relu=False)
    return b.done(), False


def chain_from_depthwise(B, T):
    b = _Builder("chain_from_depthwise", 92, B, 512, T)
    b.op("dw", 512, k=31, groups=512, relu=False)
    b.op("up", 1024)
    b.op("down", 512, relu=False)
    return b.done(), False


def projection_and_pair(B, T):
    b = _Builder("projection_and_pair", 92, B, 256, T)
    b.op("proj", 256, relu=False, advance=False)          # (of which nobody reads the output)
    b.op("dw", 256, k=33, groups=256, relu=False)
    b.op("pw", 256)
    return b.done(), True


@pytest.mark.parametrize("net", [pair, chain, chain_from_depthwise, projection_and_pair])
@pytest.mark.parametrize("B,T,off", [(1, 96, 0), (2, 160, 0), (3, 160, 16 * 37), (2, 99, 0), (1, 61, 64 * 61)])
def test_output_over_input(net, B, T, off, tuning_env):
    tuning_env("QASR_PW_CHAIN", "1")
    net, always_workspace = net(B, T)
    params = W.draw_net_params(net, 5)
    x = W.draw_input(net, 5)
    ref = oracle.encoder_forward(net, params, x)
    g = GpuNet(net, params)
    print(f"[case] {net.name} B={B} T={T} off={off}", flush=True)
    assert np.array_equal(g.forward(dev(x)).cpu().numpy(), ref)
    if T % 16 == 0:
        assert {g.enc.op_launch(i)[0] for i in range(g.enc.n_ops)} == {0}     # all layers in one launch ...
        assert always_workspace or bool((g.ws == FILL).all())                 # ... which needs no tensor between them
    n = x.size
    raw = torch.full((n + off,), FILL, dtype=torch.int8, device="cuda")
    xd, yd = raw[:n].view(x.shape), raw[off:].view(ref.shape)

    def again():
        raw.fill_(FILL)
        xd.copy_(torch.from_numpy(x))
        g.ws.fill_(FILL)
    again()
    g.enc.forward(xd, yd, g.ws)
    assert np.array_equal(yd.cpu().numpy(), ref)
    if not always_workspace:
        assert not bool((g.ws == FILL).all())                                 # launches of their own
    again()
    graph = g.enc.graph(xd, yd, g.ws)
    for _ in range(3):
        again()
        graph.launch()
        assert np.array_equal(yd.cpu().numpy(), ref)
    if g.enc.workspace_bytes <= 32 << 20:
        again()
        g.enc.forward_static(xd, yd)
        assert np.array_equal(yd.cpu().numpy(), ref)
    g.check_guards()
    graph.close()
    g.enc.close()


def test_layers_that_only_write_the_output_keep_their_launch(tuning_env):
    """A chain that ends at the network's output but does not read its input stays one launch."""
    tuning_env("QASR_PW_CHAIN", "1")
    b = _Builder("later_chain", 92, 2, 64, 80)
    b.op("in", 512)
    b.op("up", 1024)
    b.op("down", 512, relu=False)
    b.op("up2", 1024, relu=False)
    net = b.done()
    params = W.draw_net_params(net, 6)
    x = W.draw_input(net, 6)
    g = GpuNet(net, params)
    raw = torch.zeros(net.B * net.Cout * net.Tout, dtype=torch.int8, device="cuda")
    xd = raw[:x.size].view(x.shape)
    xd.copy_(torch.from_numpy(x))
    yd = raw.view(net.B, net.Cout, net.Tout)
    ms = g.enc.forward_timed(xd, yd, g.ws)
    assert ms[2] == 0.0 and ms[3] == 0.0
    xd.copy_(torch.from_numpy(x))
    g.enc.forward(xd, yd, g.ws)
    assert np.array_equal(yd.cpu().numpy(), oracle.encoder_forward(net, params, x))
    g.enc.close()
