"""The rescale of GLU (csrc/act.hip) on both sides of s = 33, over every pair of codes: one piece per thread, several, and
the scalar tail."""
import numpy as np
import pytest
import torch

import oracle
import paper_2103_16827_amd as Q
from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,extra", [(1, 0), (2, 1)])
@pytest.mark.parametrize("m", [0, 1, 1 << 30, (1 << 31) - 1])
@pytest.mark.parametrize("s", [1, 20, 32, 33, 34, 45, 52, 62])
def test_glu_rescale(s, m, B, extra):
    T = 256 + extra                                     # (257: halves off the 16-byte grid)
    x = np.zeros((B, 512, T), np.int8)                  # value c - 128 against every gate code
    x[:, :256] = (np.arange(256) - 128).reshape(256, 1)
    x[:, 256:, :256] = (np.arange(256) - 128).reshape(1, 256)
    print(f"[case] GLU m={m} s={s} B={B} T={T}", flush=True)
    y = torch.empty((B, 256, T), dtype=torch.int8, device="cuda")
    Q.act_int8(Q.make_act(Q.ACT_GLU, Q.iexp_init(5.0 / 127, 8), m, s), dev(x), B, 256, T, y, 512 * T, 256 * T)
    ref = oracle.act(Q.ACT_GLU, x, oracle.iexp_constants(5.0 / 127, 8), m, s)
    assert np.array_equal(y.cpu().numpy(), ref)


def test_several_pieces_per_thread():
    B, C, T = 1024, 64, 400                             # (more pieces than the launch has threads)
    rng = np.random.default_rng(4)
    x = rng.integers(-128, 128, (B, 2 * C, T), dtype=np.int8)
    y = torch.empty((B, C, T), dtype=torch.int8, device="cuda")
    Q.act_int8(Q.make_act(Q.ACT_GLU, Q.iexp_init(5.0 / 127, 8), 1 << 30, 45), dev(x), B, C, T, y, 2 * C * T, C * T)
    ref = oracle.act(Q.ACT_GLU, x, oracle.iexp_constants(5.0 / 127, 8), 1 << 30, 45)
    assert np.array_equal(y.cpu().numpy(), ref)
