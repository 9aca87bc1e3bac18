"""The 16-wave pointwise kernel (csrc/pw_wide.hip): every tile and split of the input channels, ragged rows and
channels, residual, both clamps, the 64-bit rescale, batch strides, an activation's table; the edges of
its widths."""
import pytest

import paper_2103_16827_amd as Q
import qasr_workloads as W
from gpu_util import desc_of, dev, Guarded, GpuNet
from qasr_workloads.nets import _Builder
import numpy as np
import torch
import oracle
from test_gpu_parity import layer_case, run_layer_case

pytestmark = pytest.mark.gpu


def run_wide(case, extra=None):
    op, _, x, _, _ = case
    d = desc_of(op, x.shape[0], Q.FLAG_W_PACKED)
    d.y_batch_stride = 0 if extra is None else op.Cout * op.Tout + extra
    assert Q.conv1d_launch_name(d) == "pw_wide"
    run_layer_case(case, extra)


TILES = ["1,1", "2,1", "4,1", "7,1", "1,2", "2,2", "4,2", "7,2", "1,4", "2,4", "4,4", "1,8", "2,8", "4,8"]
SHAPES = [
    dict(name="w512_res", B=2, Cin=512, Cout=512, T=176, res=True, packed=True),
    dict(name="w384_ragged", B=3, Cin=384, Cout=200, T=75, res=True, relu=False, packed=True),
    dict(name="w960_29", B=2, Cin=960, Cout=29, T=112, relu=False, bias=False, packed=True),
    dict(name="w64_1000", B=5, Cin=64, Cout=1000, T=31, packed=True, s_lo=20, s_hi=40),
]


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("kw", SHAPES, ids=[c["name"] for c in SHAPES])
def test_tiles(kw, tile, tuning_env):
    if kw["Cin"] // 64 < int(tile.split(",")[1]):
        pytest.skip("fewer 64-channel chunks than groups")
    tuning_env("QASR_PW_WIDE", "1")
    tuning_env("QASR_PWW", tile)
    print(f"[case] tile {tile}", flush=True)
    run_wide(layer_case(**kw))


@pytest.mark.parametrize("extra", [16, 4])
@pytest.mark.parametrize("kw", [dict(name="w2048", B=2, Cin=2048, Cout=256, T=48, packed=True),
                                dict(name="w1024_T5", B=9, Cin=1024, Cout=96, T=5, packed=True, res=True),
                                dict(name="w128_T4", B=40, Cin=128, Cout=16, T=4, packed=True),
                                dict(name="w512_T1", B=3, Cin=512, Cout=512, T=1601, packed=True)], ids=lambda k: k["name"])
def test_edges_and_batch_strides(kw, extra, tuning_env):
    tuning_env("QASR_PW_WIDE", "1")
    run_wide(layer_case(**kw), extra)


@pytest.mark.parametrize("B,T,stride", [(3, 48, 1 << 28), (3, 48, 1 << 30), (8, 16, 1 << 28), (9, 16, 1 << 29), (2, 112, (1 << 31) + 64), (2, 31, (1 << 31) + 1)])
def test_items_far_apart(B, T, stride):
    """A view whose batch items lie so far apart that a tile's offsets do or do not fit 32 bits."""
    op, p, x, _, _ = layer_case("w_far", B, 192, 80, T, packed=True)
    d = desc_of(op, B)
    d.x_batch_stride = stride
    wp = torch.empty(Q.packed_weight_bytes(d), dtype=torch.int8, device="cuda")
    Q.pack_weights(d, dev(p["w"]), wp)
    d.flags |= Q.FLAG_W_PACKED
    assert Q.conv1d_launch_name(d) == "pw_wide"
    n = op.Cin * T
    far = torch.empty((B - 1) * stride + n, dtype=torch.int8, device="cuda")
    for b in range(B):
        far[b * stride:b * stride + n] = dev(x[b]).reshape(-1)
    y = Guarded(B * op.Cout * T)
    print(f"[case] {B} items {stride} bytes apart, T={T}", flush=True)
    Q.conv1d_int8(d, far, wp, dev(p["bias"]), dev(p["m"]), dev(p["s"]), None, y.view)
    torch.cuda.synchronize()
    y.check()
    assert np.array_equal(y.view.cpu().numpy().reshape(B, op.Cout, T), oracle.run_op(op, p, x))


@pytest.mark.parametrize("T", [80, 61])
def test_activation_table(T, tuning_env):
    tuning_env("QASR_PW_WIDE", "1")
    b = _Builder("wide_act", 91, 3, 192, T)
    t1 = b.op("p1", 320, relu=False, act=2)
    b.op("p2", 320, relu=True, res=t1, act=1)
    b.op("p3", 128, relu=False, act=2)
    net = b.done()
    params = W.draw_net_params(net, 2)
    x = W.draw_input(net, 2)
    g = GpuNet(net, params)
    print(f"[case] activations in pw_wide, kernels {[g.enc.op_launch(i) for i in range(3)]}", flush=True)
    assert [g.enc.op_launch(i) for i in range(3)] == [(i, "pw_wide") for i in range(3)]
    assert [g.enc.op_act_fused(i) for i in range(3)] == [True, True, True]
    assert np.array_equal(g.forward(dev(x)).cpu().numpy(), oracle.encoder_forward(net, params, x))
    g.check_guards()
    g.enc.close()
