"""Dense layers at the edges of conv_pipe's rounds: 1, 2 and 3 steps past whole rounds of four, fewer steps than
a round, two and three taps per chunk (a chunk is committed while its successor is on its way), rows that end
inside a four-frame unit, for every tile height.  The dense shapes of the networks, which conv_few runs at these
sizes, in the tile that conv_pipe chooses by itself, with and without gaps between the batch items' blocks."""
import pytest

import paper_2103_16827_amd as Q
from gpu_util import desc_of
from test_gpu_parity import DENSE, STRIDED, layer_case, run_layer_case

pytestmark = pytest.mark.gpu

SHAPES = [
    dict(name="two_steps", B=1, Cin=64, Cout=64, T=16, k=2, packed=True),
    dict(name="k2_chunks5", B=1, Cin=320, Cout=130, T=323, k=2, packed=True, s_lo=20, s_hi=44),
    dict(name="k3_chunks3", B=2, Cin=192, Cout=128, T=161, k=3, packed=True, res=True),
    dict(name="k7_chunks2_d3", B=2, Cin=128, Cout=256, T=145, k=7, dil=3, packed=True, relu=False),
    dict(name="k11_chunks3", B=1, Cin=192, Cout=192, T=330, k=11, packed=True, bias=False),
]


@pytest.mark.parametrize("tile", ["4,2,1", "5,2,1", "9,2,1", "10,2,1", "5,4,1", "7,4,1", "8,2,2", "10,2,2"])
@pytest.mark.parametrize("kw", SHAPES, ids=[c["name"] for c in SHAPES])
def test_rounds(kw, tile, tuning_env):
    tuning_env("QASR_CP_TILE", tile)
    assert run_layer_case(layer_case(**kw)) == "conv_pipe"


NETWORKS = DENSE + [c for c in STRIDED if c.get("k", 1) > 1 and not c.get("dw") and c.get("packed")]


@pytest.mark.parametrize("extra", [None, 16, 4])
@pytest.mark.parametrize("kw", NETWORKS, ids=[c["name"] for c in NETWORKS])
def test_without_conv_few(kw, extra, tuning_env):
    tuning_env("QASR_NO_CONV_FEW", "1")
    case = layer_case(**kw)
    assert Q.conv1d_launch_name(desc_of(case[0], kw["B"], Q.FLAG_W_PACKED)) == "conv_pipe"
    run_layer_case(case, extra)
