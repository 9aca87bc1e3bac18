"""Integer softmax at the edges of its lane-group sizes and of the range its 32-bit form takes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2103_16827_amd as Q
from qasr_workloads.rng import randint_array

pytestmark = pytest.mark.gpu

# (scale, u): the usual one; exponentials just below and above 2^24; 2^u > q_ln2; small q_ln2
SCALES = [(0.01, 2), (0.00041, 0), (0.00039, 0), (0.9, 3), (0.02, 0), (1.3, 6)]


@pytest.mark.parametrize("L", [1, 3, 16, 17, 32, 33, 64, 65, 127, 128, 129, 256, 257, 400, 511, 512, 513, 1023, 1024,
                               1025, 2048, 2049, 4095, 4096, 4097])
@pytest.mark.parametrize("rows", [5, 4001])
def test_softmax_sizes(rows, L):
    rows = min(rows, max(5, (1 << 21) // L))
    for S, u in SCALES:
        print(f"[case] softmax rows={rows} L={L} S={S} u={u}", flush=True)
        x = randint_array(7 + L, (rows, L), -int(4 / S), int(4 / S) + 1, np.int32)
        x[0, :] = np.iinfo(np.int32).min
        x[1, :] = np.iinfo(np.int32).min
        x[1, L // 2] = np.iinfo(np.int32).max
        x[2, :] = np.iinfo(np.int32).min + 1         # equal quotients
        if L > 1:
            x[3, :] = -int(40 / S)
            x[3, :2] = 0                             # two halves: quotients on whole numbers
        ref = oracle.softmax(x, oracle.iexp_constants(S, u))
        xd = torch.from_numpy(x).cuda()
        yd = torch.full((rows * L + 16,), 99, dtype=torch.int8, device="cuda")
        Q.softmax_int32(Q.iexp_init(S, u), xd, yd[: rows * L].view(rows, L))
        torch.cuda.synchronize()
        got = yd.cpu().numpy()
        assert np.array_equal(got[: rows * L].reshape(rows, L), ref)
        assert np.all(got[rows * L:] == 99)


def test_more_rows_than_one_grid_dimension():
    """2^30 - 3 rows: one lane group per row is more than 2^32 work items along one dimension of a grid."""
    rows, L, S, u = (1 << 30) - 3, 2, 0.01, 2
    print(f"[case] softmax rows={rows} L={L}", flush=True)
    period = 1 << 12
    x = randint_array(11, (period, L), -400, 401, np.int32)
    ref = torch.from_numpy(oracle.softmax(x, oracle.iexp_constants(S, u))).cuda()
    xd = torch.from_numpy(x).cuda().repeat(-(-rows // period), 1)
    yd = torch.full((rows + 16, L), 99, dtype=torch.int8, device="cuda")
    Q.softmax_int32(Q.iexp_init(S, u), xd[:rows], yd[:rows])
    torch.cuda.synchronize()
    whole = rows // period
    assert bool((yd[: whole * period].view(whole, period, L) == ref).all())
    assert bool((yd[whole * period: rows] == ref[: rows - whole * period]).all())
    assert bool((yd[rows:] == 99).all())
