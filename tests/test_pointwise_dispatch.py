"""Which pointwise layers pw_wide takes from the families of the benchmark's widths, on either side of each line
(host only), and those families' own kernels on all the layer cases, since small launches go to pw_wide."""
import pytest

import paper_2103_16827_amd as Q
from paper_2103_16827_amd.binding import make_desc
from gpu_util import desc_of
from test_gpu_parity import PIPE, REAL, STRIDED, layer_case, run_layer_case


def launched(Cin, Cout, G, B=2):
    return Q.conv1d_launch_name(make_desc(B, Cin, Cout, 16 * G // B, flags=Q.FLAG_W_PACKED))


@pytest.mark.parametrize("Cin,Cout,last", [(640, 768, 896), (384, 1500, 594), (384, 200, 128), (640, 29, 640), (1024, 29, 700), (2048, 512, 200), (1024, 1024, 50),
                                           (1024, 256, 200), (512, 768, 294), (512, 1000, 800), (256, 384, 200)])
def test_launches_up_to_a_line(Cin, Cout, last):
    assert launched(Cin, Cout, last) == "pw_wide"
    assert launched(Cin, Cout, last + 2) in ("pw_pipe", "pw_tile")


@pytest.mark.parametrize("Cin,Cout,wide", [(384, 512, True), (1024, 1000, True), (256, 128, False), (512, 512, False), (512, 2048, False)])
@pytest.mark.parametrize("G", [2, 200, 1400, 3200])
def test_shapes_with_one_choice(Cin, Cout, wide, G):
    assert (launched(Cin, Cout, G) == "pw_wide") == wide


@pytest.mark.parametrize("B,Cin,T,stride", [(4, 64, 1 << 22, 0), (1, 2048, 1 << 21, 0), (64, 64, 1 << 22, 0), (2, 64, 32, 1 << 33),
                                            (40, 64, 16, 1 << 29), (2, 64, 33, 1 << 31)])
def test_large_inputs_keep_the_kernel(B, Cin, T, stride):
    """Items of 256 MiB and more, and views whose items lie far apart."""
    assert Q.conv1d_launch_name(make_desc(B, Cin, 16, T, x_batch_stride=stride, flags=Q.FLAG_W_PACKED)) == "pw_wide"


POINTWISE = [c for c in PIPE + REAL + STRIDED if c.get("k", 1) == 1 and c.get("packed")]


@pytest.mark.gpu
@pytest.mark.parametrize("extra", [None, 16, 4])
@pytest.mark.parametrize("kw", POINTWISE, ids=[c["name"] for c in POINTWISE])
def test_without_pw_wide(kw, extra, tuning_env):
    tuning_env("QASR_NO_PW_WIDE", "1")
    case = layer_case(**kw)
    op, _, x, _, _ = case
    d = desc_of(op, x.shape[0], Q.FLAG_W_PACKED)
    d.y_batch_stride = 0 if extra is None else op.Cout * op.Tout + extra
    assert Q.conv1d_launch_name(d) == Q.conv1d_kernel_name(d) != "pw_wide"
    run_layer_case(case, extra)


@pytest.mark.gpu
def test_without_pw_wide_reaches_the_families(tuning_env):
    tuning_env("QASR_NO_PW_WIDE", "1")
    seen = set()
    for kw in POINTWISE:
        op, _, x, _, _ = layer_case(**kw)
        seen.add(Q.conv1d_launch_name(desc_of(op, x.shape[0], Q.FLAG_W_PACKED)))
    assert seen == {"pw_pipe", "pw_tile", "gemm_mfma"}
