"""Shifts above the short rescale's range with a residual (54 < s) and up to the largest one, in the pointwise
kernels: biases up to 2^30 in size, so that the rescaled value is not just 0."""
import numpy as np
import pytest

from qasr_workloads.rng import randint_array
from test_gpu_parity import layer_case, run_layer_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("relu", [True, False])
@pytest.mark.parametrize("res", [True, False])
@pytest.mark.parametrize("form", ["pipe", "lean", "wide"])
@pytest.mark.parametrize("lo,hi", [(50, 62), (55, 62)])
def test_large_shifts(lo, hi, form, res, relu, tuning_env):
    if form == "pipe":
        tuning_env("QASR_NO_PW_WIDE", "1")
    if form == "lean":
        tuning_env("QASR_PW_LEAN", "1")
    if form == "wide":
        tuning_env("QASR_PW_WIDE", "1")
    Cout = 512 if form == "lean" else 768                # (passes that are pipelined and a last one that is not)
    op, p, x, r, packed = layer_case(name=f"s_{lo}_{hi}_{form}", B=2, Cin=256, Cout=Cout, T=176, s_lo=lo, s_hi=hi,
                                     res=res, relu=relu, packed=True)
    p["bias"] = randint_array(17, (Cout,), -(1 << 30), 1 << 30, np.int32)
    if lo > 54:                                          # one pass of short shifts between the others
        p["s"][256:512] = randint_array(18, (256,), 33, 55, np.int32)
    run_layer_case((op, p, x, r, packed))
