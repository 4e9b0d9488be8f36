"""The two-level bucket sort gives bitwise the grids of the atomic one at the
sizes where its launch changes: workgroup counts (with and without the column
scan), super-bucket edges, one workgroup per super-bucket or a counter."""

import numpy as np
import pytest

from gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu


# particles: 1; one and two workgroups; 16 (no column scan) and 17; grids: super-bucket
# edges of 2 (24), 4 (64), 5 (100); the bucket pass with more super-buckets
# than workgroups (128); orders 5 and 6 keep the longer edges
@pytest.mark.parametrize("n_grid,order,n,sets,dtype", [
    (24, 4, 1, 1, np.float32), (24, 2, 4096, 1, np.float32), (24, 3, 4097, 3, np.float64),
    (64, 4, 65536, 1, np.float32), (64, 4, 65537, 1, np.float64), (64, 6, 65537, 2, np.float32),
    (100, 3, 70001, 5, np.float32), (100, 5, 30000, 1, np.float32), (128, 1, 300000, 2, np.float32),
])
@pytest.mark.parametrize("weighted", [False, True])
def test_two_level_equals_atomic(n_grid, order, n, sets, dtype, weighted):
    torch = require_gpu()
    from paper_1512_07295_amd.estimator import Estimator

    box = 300.0
    rng = np.random.default_rng(n + order)
    pos = rng.uniform(0, box, (n, 3))
    pos[: n // 3] = np.mod(rng.normal(0.2 * box, 0.02 * box, (n // 3, 3)), box)
    pos = to_dev(torch, pos[rng.permutation(n)].astype(dtype))
    w = to_dev(torch, rng.exponential(1.0, n).astype(np.float32)) if weighted else None
    offs = None
    if sets > 1:
        offs = to_dev(torch, np.linspace(0, n, sets + 1).astype(np.int64))
    grids, powers = [], []
    for atomic in (False, True):
        est = Estimator(n_grid, box, order, 1, sets, n, atomic_sort=atomic, weighted=weighted)
        if weighted:
            est.set_weights(w)
        est.deposit(pos, offs)
        grids.append([est.copy_grid(g, m).cpu() for m in range(sets) for g in (1, 2)])
        powers.append(est.power(pos, offs, subtract_shot=True)[1].cpu())
        est.close()
    for a, b in zip(*grids):
        assert torch.equal(a, b)
    assert torch.allclose(powers[0], powers[1], rtol=1e-12, atol=0, equal_nan=True)
