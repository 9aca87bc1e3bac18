"""Pairs of a depthwise and a pointwise layer in tiles of one and two groups (csrc/sep_body.hpp, sep_small_kernel):
weight rows permuted into Toeplitz form for every shift of the first tap (r = 0 .. 3) and dilations, one to nine
chunks per row, partial last groups and tiles, every split of the pointwise half over the waves, caller's rows at any address."""
import pytest

import qasr_workloads as W
from test_sep_gpu import chain, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", ["1,1", "1,1,2", "1,2", "2,1", "2,1,2", "2,2"])
@pytest.mark.parametrize("C,Cout,k,dil,T,opt", [
    (256, 512, 1, 1, 33, dict()), (256, 512, 6, 1, 64, dict(res=True)), (512, 512, 33, 1, 49, dict(res=True, act=2)),
    (512, 512, 39, 2, 96, dict(dw_bias=True)), (256, 512, 61, 1, 31, dict(dw_relu=True, dw_bias=True)),
    (512, 512, 87, 1, 130, dict(act=1, pw_relu=False)), (256, 512, 29, 3, 16, dict(res=True))],
    ids=lambda v: str(v).replace(" ", ""))
def test_small_tiles(C, Cout, k, dil, T, opt, tile, tuning_env):
    print(f"[case] sep {C}->{Cout} k={k} dil={dil} T={T} {opt} tile {tile}", flush=True)
    tuning_env("QASR_SEP", tile)
    check(chain(2, T, C, Cout, k, dil=dil, **opt))


@pytest.mark.parametrize("tile", ["1,1,2", "2,1,2"])
@pytest.mark.parametrize("T", [5, 203])
def test_pair_is_the_whole_encoder(T, tile, tuning_env):
    print(f"[case] separable module T={T} tile {tile}", flush=True)
    tuning_env("QASR_SEP", tile)
    check(W.separable_module(2, 256, T, 33))


@pytest.mark.parametrize("lo,hi", [(20, 40), (54, 62)])
def test_rescale_ranges(lo, hi, tuning_env):
    print(f"[case] sep s in {lo}..{hi}", flush=True)
    tuning_env("QASR_SEP", "2,1,2")
    check(chain(1, 40, 256, 256, 33, res=True), s_lo=lo, s_hi=hi)
