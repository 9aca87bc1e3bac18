"""Encoders whose utterance lengths are not multiples of 16 frames: the library keeps its own tensors in
rows rounded up to 16, whose pad bytes hold arbitrary values (the workspace starts as a fill pattern
here).  Lengths around the edges of a 16-frame chunk and of a dword, batches that take either
depthwise kernel, the int8 and the float entry, against the oracle byte for byte."""
import numpy as np
import pytest
import torch

import oracle
import qasr_workloads as W
from gpu_util import dev, GpuNet
from qasr_workloads.nets import _Builder

pytestmark = pytest.mark.gpu

NETS = {
    "quartznet": lambda B, T: W.quartznet(B, T, 1, 1, widths=(256, 256, 512), kernels=(33, 39, 75)),
    "conformer": lambda B, T: W.conformer_shaped(B, T, 4, d_model=256, d_ff=512, layers=2, nonlinear=True),
    "jasper_dr": lambda B, T: W.jasper(B, T, 3, widths=(64, 128), kernels=(11, 13), C_epi=64, k_epi=5, C_epi2=128,
                                       dense_residual=True),
    "module": lambda B, T: W.separable_module(B, 256, T, 33),
    # the last op has a residual operand: rows stay dense
    "residual_last": lambda B, T: W.NetSpec("cut", 1, B, 64, T, W.quartznet(B, T, 1, 1).ops[:12], 16),
}


@pytest.mark.parametrize("net,B,T", [
    ("quartznet", 1, 33), ("quartznet", 2, 130), ("quartznet", 13, 97), ("quartznet", 1, 2203),
    ("conformer", 1, 17), ("conformer", 3, 30), ("conformer", 12, 61),
    ("jasper_dr", 2, 31), ("jasper_dr", 1, 203),
    ("module", 1, 201), ("module", 14, 47), ("module", 1, 5), ("module", 2, 3), ("residual_last", 2, 99)])
def test_encoders_on_utterances_of_any_length(net, B, T):
    print(f"[case] {net} B={B} T={T}", flush=True)
    spec = NETS[net](B, T)
    params = W.draw_net_params(spec, 5)
    x = W.draw_input(spec, 5)
    ref = oracle.encoder_forward(spec, params, x)
    g = GpuNet(spec, params)
    for _ in range(2):                               # (the second run finds the first one's pads)
        got = g.forward(dev(x)).cpu().numpy()
        bad = np.argwhere(got != ref)
        assert bad.size == 0, f"{len(bad)} of {ref.size} differ, first at {bad[0]}, kernels {set(g.kernels())}"
    g.check_guards()
    if T >= 16:
        assert "conv_generic" not in g.kernels() or net == "residual_last"
    alpha, S = 3.0, 0.125
    xf = (x.astype(np.float32) * np.float32(alpha / 127))
    want = oracle.dequantize(oracle.encoder_forward(spec, params, oracle.quantize(xf, alpha)), S)
    ws = torch.full((g.enc.workspace_bytes_f32,), 77, dtype=torch.int8, device="cuda")
    y = torch.full(ref.shape, 77.0, dtype=torch.float32, device="cuda")
    g.enc.forward_f32(torch.from_numpy(xf).cuda(), alpha, S, y, ws)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy().view(np.uint32), want.view(np.uint32))
    g.enc.close()


@pytest.mark.parametrize("C", [384, 640])
def test_activation_at_both_ends_of_a_float_forward(C):
    """The first and the last layer are pointwise layers with a unary activation: the float entry runs them on
    padded rows, the int8 entry on the caller's dense ones, which may be another kernel's.  Each applies the
    activation once."""
    print(f"[case] activations at both ends C={C}", flush=True)
    b = _Builder("act_ends", 91, 2, C, 61)
    b.op("first", 4 * C, relu=False, act=2)
    b.op("mid", C, relu=False)
    b.op("last", 4 * C, relu=False, act=1)
    spec = b.done()
    params = W.draw_net_params(spec, 6)
    x = W.draw_input(spec, 6)
    g = GpuNet(spec, params)
    assert np.array_equal(g.forward(dev(x)).cpu().numpy(), oracle.encoder_forward(spec, params, x))
    alpha, S = 3.0, 0.125
    xf = (x.astype(np.float32) * np.float32(alpha / 127))
    want = oracle.dequantize(oracle.encoder_forward(spec, params, oracle.quantize(xf, alpha)), S)
    ws = torch.full((g.enc.workspace_bytes_f32,), 77, dtype=torch.int8, device="cuda")
    y = torch.full(want.shape, 77.0, dtype=torch.float32, device="cuda")
    g.enc.forward_f32(torch.from_numpy(xf).cuda(), alpha, S, y, ws)
    torch.cuda.synchronize()
    bad = np.argwhere(y.cpu().numpy() != want)
    assert bad.size == 0, f"{len(bad)} of {want.size} differ, first at {bad[0]}"
    g.enc.close()
