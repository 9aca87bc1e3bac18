"""Dense layers of few frames (csrc/conv_few.hip): every tile, fewer steps than wave groups and more than rings, taps that
wrap over several chunks per step, ragged rows and channels, strides, dilations, several residual operands, a transposition unit
for every thread and for fewer than a wave; the choice the library makes for small encoders, replayed as a graph."""
import numpy as np
import pytest
import torch

import oracle
import paper_2103_16827_amd as Q
import qasr_workloads as W
from gpu_util import GpuNet, desc_of, dev, gpu_layer
from qasr_workloads.nets import _Builder
from test_gpu_parity import draw, layer_case, run_layer_case

pytestmark = pytest.mark.gpu

SHAPES = [
    dict(name="k2_one_chunk", B=1, Cin=64, Cout=64, T=16, k=2, packed=True),
    dict(name="k3_chunks5", B=2, Cin=320, Cout=130, T=67, k=3, packed=True, s_lo=20, s_hi=44),
    dict(name="k11_res", B=2, Cin=256, Cout=256, T=101, k=11, packed=True, res=True, relu=False),
    dict(name="k13_s2", B=1, Cin=128, Cout=200, T=150, k=13, stride=2, pad=(6, 6), packed=True, bias=False),
    dict(name="k29_d2", B=1, Cin=768, Cout=96, T=130, k=29, dil=2, packed=True),
    dict(name="k5_T4", B=3, Cin=192, Cout=64, T=4, k=5, packed=True),
]


def takes_few(op, B):
    """The kernel that the call launches (a layer's kernel name is its family's, conv_pipe, for both)."""
    return Q.conv1d_launch_name(desc_of(op, B, Q.FLAG_W_PACKED)) == "conv_few"


@pytest.mark.parametrize("tile", ["1,1", "2,1", "3,1", "4,1", "1,2", "2,2", "3,2", "4,2"])
@pytest.mark.parametrize("kw", SHAPES, ids=[c["name"] for c in SHAPES])
def test_tiles(kw, tile, tuning_env):
    tuning_env("QASR_CONV_FEW", "1")
    tuning_env("QASR_CF", tile)
    case = layer_case(**kw)
    assert takes_few(case[0], kw["B"])
    run_layer_case(case)


@pytest.mark.parametrize("tile", ["1,1,1", "2,1,1", "3,1,1", "4,1,1", "1,1,3", "2,1,3", "3,1,3", "4,1,3"])
@pytest.mark.parametrize("kw", SHAPES, ids=[c["name"] for c in SHAPES])
def test_tiles_of_16_and_48_channels(kw, tile, tuning_env):
    test_tiles(kw, tile, tuning_env)


@pytest.mark.parametrize("T", [4, 5, 7, 8, 9, 15, 17, 23])
def test_rows_about_eight_frames_long(T, tuning_env):
    """A unit of eight frames over a row's end, over both rows' ends, and rows that are shorter than one."""
    tuning_env("QASR_CONV_FEW", "1")
    for B, Cin, pad in ((1, 64, (1, 1)), (2, 128, (0, 2)), (3, 64, (13, 13))):
        k = pad[0] + pad[1] + 1
        print(f"[case] dense {Cin} -> 64 k={k} B={B} T={T}", flush=True)
        case = layer_case("few_frames", B, Cin, 64, T, k=k, pad=pad, packed=True)
        assert takes_few(case[0], B)
        run_layer_case(case)


@pytest.mark.parametrize("B,Cin,T,k,dil,pad,units", [(1, 1024, 20, 15, 7, (49, 49), 1024), (2, 64, 25, 14, 7, (45, 46), 60)])
def test_units_for_all_threads_and_for_less_than_a_wave(B, Cin, T, k, dil, pad, units, tuning_env):
    """A unit is 8 rows of LDS x 16 channels, one per thread at most: 160 KiB hold 1024."""
    tuning_env("QASR_CONV_FEW", "1")
    tuning_env("QASR_CF", "1,1,1")
    assert units == Cin // 64 * ((15 + dil * (k - 1) + 1 + 7 + 7) // 8 * 8) // 2
    case = layer_case("few_units", B, Cin, 64, T, k=k, dil=dil, pad=pad, packed=True)
    assert takes_few(case[0], B)
    run_layer_case(case)


@pytest.mark.parametrize("n_res", [2, 5, 12])
def test_several_residuals(n_res, tuning_env):
    tuning_env("QASR_CONV_FEW", "1")
    op, p, x, _, packed = layer_case("few_res", 2, 256, 192, 77, k=11, packed=True)
    assert takes_few(op, 2)
    rs = [draw(55 + r, (2, op.Cout, op.Tout), -128, 127, np.int8) for r in range(n_res)]
    print(f"[case] dense 256 -> 192 k=11 with {n_res} residuals", flush=True)
    assert np.array_equal(gpu_layer(op, 2, p, x, rs, packed=packed), oracle.run_op(op, p, x, rs))


@pytest.mark.parametrize("B,T", [(1, 60), (2, 211)])
def test_small_encoder_takes_it(B, T):
    net = W.jasper(B, T, 3, widths=(256, 512), kernels=(11, 17), per_width=1, C_epi=320, k_epi=29, C_epi2=128)
    params, x = W.draw_net_params(net, 8), W.draw_input(net, 8)
    print(f"[case] small Jasper B={B} T={T}", flush=True)
    ref = oracle.encoder_forward(net, params, x)
    g = GpuNet(net, params)
    assert "conv_few" in [g.enc.op_launch(i)[1] for i in range(g.enc.n_ops)]
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


@pytest.mark.parametrize("C,k,B,T,splits", [(768, 25, 4, 400, True), (768, 25, 2, 800, True), (256, 11, 2, 406, False),
                                            (768, 25, 1, 104, False)])
def test_the_kernel_named_is_the_one_that_runs(C, k, B, T, splits):
    """Between the two dense kernels the forward chooses with the room that it has for partial sums; what is written there tells
    whether conv_pipe ran in several parts (the room is the largest such layer's: without one there is none)."""
    b = _Builder("two_layers", 91, B, 64, T)
    b.op("in", C)
    b.op("dense", C, k=k)
    net = b.done()
    g = GpuNet(net, W.draw_net_params(net, 8))
    pitch = (T + 15) // 16 * 16
    slot, counters = (B * C * pitch + 255) // 256 * 256, 4096
    room = g.enc.workspace_bytes - slot - counters
    print(f"[case] {C} -> {C} k={k} B={B} T={T}: {g.enc.op_launch(1)}, room {room}", flush=True)
    g.ws.fill_(77)
    g.forward(dev(W.draw_input(net, 8)))
    torch.cuda.synchronize()
    ran_in_parts = room > 0 and bool((g.ws[slot:slot + room] != 77).any())
    assert ran_in_parts == splits
    assert g.enc.op_launch(1) == (1, "conv_pipe" if ran_in_parts else "conv_few")
    g.check_guards()
    g.enc.close()
