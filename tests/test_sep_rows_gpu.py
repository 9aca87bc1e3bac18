"""How pairs of a depthwise and a pointwise layer bring in their rows (csrc/sep_body.hpp): a caller's rows shorter than the 16 bytes
of a load, the tensor's last rows, frames past a row's end in every chunk of a tile's rows, and more than eight chunks per row
(sixteen lanes bring one in)."""
import pytest

import qasr_workloads as W
from qasr_workloads.nets import _Builder
from test_sep_gpu import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", ["1,1,2", "2,1", "4,1"])
@pytest.mark.parametrize("T", [4, 15, 16, 17, 31, 61])
def test_rows_of_the_caller(T, tile, tuning_env):
    print(f"[case] separable module T={T} tile {tile}", flush=True)
    tuning_env("QASR_SEP", tile)
    check(W.separable_module(3, 256, T, 33))


@pytest.mark.parametrize("tile", ["1,1,2", "2,1,2", "2,1", "7,1"])
@pytest.mark.parametrize("C,T", [(256, 97), (512, 144), (512, 175)])
def test_nine_chunks_per_row(C, T, tile, tuning_env):
    print(f"[case] sep {C} k=87 padded 33 | 53, T={T} tile {tile}", flush=True)
    tuning_env("QASR_SEP", tile)
    b = _Builder("sep_rows", 91, 2, 64, T)
    b.op("in", C, k=3)
    b.op("dw", C, k=87, pad=(33, 53), groups=C, relu=False, bias=False)
    b.op("pw", 256)
    b.op("out", 29, relu=False)
    check(b.done())
