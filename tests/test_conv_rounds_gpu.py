"""Dense layers at the edges of conv_pipe's rounds: 1, 2 and 3 steps past whole rounds of four, fewer steps than
a round, two and three taps per chunk (a chunk is committed while its successor is on its way), rows that end
inside a four-frame unit, for every tile height."""
import pytest

from test_gpu_parity import layer_case, run_layer_case

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
