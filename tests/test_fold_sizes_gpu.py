"""Weight folding at the edges of its register-resident forms (4 * 512 * {1, 2, 4, 8, 13} weights per
channel, longer ones read twice), with quotients on and next to rounding ties."""
import numpy as np
import pytest
import torch

import oracle
import paper_2103_16827_amd as Q
from qasr_workloads.rng import randint_array

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per", [1, 3, 2047, 2048, 2049, 4097, 8191, 16384, 16385, 26624, 26627, 30001])
def test_fold_sizes(per):
    print(f"[case] fold per={per}", flush=True)
    C = 3
    # channel 0: multiples of half a step (a tie for every odd one) when gamma / sqrt(var + eps) = 1
    w = randint_array(per, (C, per, 1), -254, 254, np.int32).astype(np.float32) * np.float32(0.5)
    w[:, 0] = 127.0
    w[1:] *= randint_array(per + 1, (C - 1, per, 1), 1 << 20, 1 << 24, np.int32).astype(np.float32) / np.float32(1 << 24)
    w[1:] = np.nextafter(w[1:], np.float32(1e9))
    one, zero = np.ones(C, np.float32), np.zeros(C, np.float32)
    gamma = np.array([1.0, 0.37, -2.5], np.float32)
    ref = oracle.fold_quantize(w, None, gamma, zero, zero, one, 0.0, 0.03, 0.05)
    d = lambda a: torch.from_numpy(a).cuda()
    qw = torch.full((C * per + 16,), 99, dtype=torch.int8, device="cuda")
    bq, m, s = (torch.full((C,), -1, dtype=torch.int32, device="cuda") for _ in range(3))
    Sw = torch.zeros(C, dtype=torch.float32, device="cuda")
    Q.fold_bn_quantize(d(w), None, d(gamma), d(zero), d(zero), d(one), 0.0, 0.03, 0.05, qw, bq, m, s, Sw)
    torch.cuda.synchronize()
    got = qw.cpu().numpy()
    assert np.array_equal(got[:-16].reshape(w.shape), ref[0]) and np.all(got[-16:] == 99)
    for a, b in zip((bq, m, s), ref[1:4]):
        assert np.array_equal(a.cpu().numpy(), b)
    assert np.array_equal(Sw.cpu().numpy().view(np.uint32), ref[4].view(np.uint32))


def test_more_channels_than_one_grid_dimension():
    """2^23 + 3 channels: a workgroup of 512 threads per channel is more than 2^32 work items along one dimension."""
    C, per, period = (1 << 23) + 3, 4, 1 << 10
    print(f"[case] fold C={C} per={per}", flush=True)
    rep = -(-C // period)
    w = torch.from_numpy(randint_array(31, (period, per), -254, 254, np.int32).astype(np.float32)).cuda()
    gamma, beta, mean, var = (torch.from_numpy(randint_array(32 + i, (period,), 1, 99, np.int32).astype(np.float32)).cuda() for i in range(4))

    def fold(n, tile):
        t = lambda a: a.repeat(*((tile,) + (1,) * (a.dim() - 1)))[:n].contiguous()
        q = torch.full((n, per), 99, dtype=torch.int8, device="cuda")
        b, m, s = (torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(3))
        Sw = torch.zeros(n, dtype=torch.float32, device="cuda")
        Q.fold_bn_quantize(t(w), None, t(gamma), t(beta), t(mean), t(var), 1e-3, 0.02, 0.03, q, b, m, s, Sw, None)
        torch.cuda.synchronize()
        return q, b, m, s, Sw

    small = fold(period, 1)
    for a, b in zip(fold(C, rep), small):
        whole = C // period * period
        assert bool((a[:whole].view(-1, *b.shape) == b).all()) and bool((a[whole:] == b[: C - whole]).all())
