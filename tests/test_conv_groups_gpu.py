"""Dense layers whose taps are split over groups of waves (csrc/conv_pipe.hip, KG > 1): uneven tap splits,
as many groups as taps, one chunk and several, ragged frames and channels, strides; several residual
operands, as many at once as fit and more, and in the kernel the library chooses for small launches.  In an encoder the chunks are split
over workgroups as well (S > 1): as many as chunks, uneven ranges, with and without groups, replays."""
import functools

import numpy as np
import pytest
import torch

import oracle
import paper_2103_16827_amd as Q
import qasr_workloads as W
from gpu_util import GpuNet, desc_of, dev, gpu_layer
from test_gpu_parity import draw, layer_case, run_layer_case

pytestmark = pytest.mark.gpu

SHAPES = [
    dict(name="k4_one_chunk", B=1, Cin=64, Cout=128, T=100, k=4, packed=True),
    dict(name="k5_ragged", B=2, Cin=192, Cout=200, T=131, k=5, packed=True, res=True, relu=False),
    dict(name="k11_wide", B=1, Cin=256, Cout=384, T=203, k=11, packed=True),
    dict(name="k13_s2", B=2, Cin=128, Cout=256, T=333, k=13, stride=2, pad=(6, 6), packed=True, bias=False),
    dict(name="k29_d2", B=1, Cin=320, Cout=72, T=97, k=29, dil=2, packed=True, s_lo=20, s_hi=40),
]


@pytest.mark.parametrize("tile", ["4,2,2", "4,2,4", "6,2,2", "4,4,2", "6,4,2"])
@pytest.mark.parametrize("kw", SHAPES, ids=[c["name"] for c in SHAPES])
def test_forced_groups(kw, tile, tuning_env):
    tuning_env("QASR_CP_TILE", tile)
    assert run_layer_case(layer_case(**kw)) == "conv_pipe"


@pytest.mark.parametrize("tile,kernel", [("", "conv_few"), ("4,2,4", "conv_pipe"), ("4,2,1", "conv_pipe"), ("10,2,2", "conv_pipe"),
                                         ("5,4,1", "conv_pipe")])
@pytest.mark.parametrize("n_res", [0, 1, 5, 12])
def test_small_launch_with_residuals(n_res, tile, kernel, tuning_env):
    """(conv_pipe asks for the rows of 6, 3, 3 and 2 operands at once in these tiles.)"""
    if tile:
        tuning_env("QASR_CP_TILE", tile)
    op, p, x, _, packed = layer_case("small", 2, 640, 640, 203, k=21, packed=True)
    assert Q.conv1d_launch_name(desc_of(op, 2, Q.FLAG_W_PACKED)) == kernel
    rs = [draw(77 + r, (2, op.Cout, op.Tout), -128, 127, np.int8) for r in range(n_res)]
    print(f"[case] dense 640 -> 640 k=21 with {n_res} residuals, tile {tile} of {kernel}", flush=True)
    ref = oracle.run_op(op, p, x, rs if n_res > 1 else (rs[0] if rs else None))
    got = gpu_layer(op, 2, p, x, rs if n_res > 1 else (rs[0] if rs else None), packed=packed)
    assert np.array_equal(got, ref)


@functools.lru_cache(maxsize=None)
def jasper_dr_case(B, T):
    net = W.jasper(B, T, 3, widths=(320, 512), kernels=(11, 4), per_width=1, C_epi=200, k_epi=5, C_epi2=128, dense_residual=True)
    params, x = W.draw_net_params(net, 9), W.draw_input(net, 9)
    return net, params, x, oracle.encoder_forward(net, params, x)


@pytest.mark.parametrize("tile", ["", "4,2,1,2", "4,2,1,5", "8,4,1,3", "7,2,1,8", "4,2,2,4", "6,4,2,2", "4,2,4,3"])
@pytest.mark.parametrize("B,T", [(1, 50), (3, 203), (2, 512)])
def test_split_contraction(B, T, tile, tuning_env):
    if tile:
        tuning_env("QASR_CP_TILE", tile)
    print(f"[case] jasper_dr B={B} T={T} tile {tile}", flush=True)
    net, params, x, ref = jasper_dr_case(B, T)
    g = GpuNet(net, params)
    assert "conv_pipe" in g.kernels()
    if tile:                                         # (the forced number of splits has its room in the workspace)
        tuning_env("QASR_CP_TILE", ",".join(tile.split(",")[:3] + ["1"]))
        whole = GpuNet(net, params)
        assert g.enc.workspace_bytes > whole.enc.workspace_bytes
        whole.enc.close()
        tuning_env("QASR_CP_TILE", tile)
    for _ in range(3):                               # (each forward finds the counters the last one left)
        assert np.array_equal(g.forward(dev(x)).cpu().numpy(), ref)
    g.check_guards()
    y = torch.zeros(ref.shape, dtype=torch.int8, device="cuda")
    ws = torch.full((max(1, g.enc.workspace_bytes),), 77, dtype=torch.int8, device="cuda")
    xd = dev(x)
    graph = g.enc.graph(xd, y, ws)
    for _ in range(3):
        y.zero_()
        graph.launch()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), ref)
        g.forward(xd)
    graph.close()
    g.enc.close()
