"""Orders 1 and 2 on sparse grids: the 16^3-tile kernel that such handles take
against the z-walking one that a handle with room for many particles takes."""

import numpy as np
import pytest

from gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu


# 256: whole tiles; 300: ragged ones
@pytest.mark.parametrize("n_grid,order,code,kind,weighted", [
    (256, 1, 0, "uniform", False), (256, 1, 1, "clump", False), (256, 2, 1, "uniform", False),
    (256, 2, 2, "uniform", True), (300, 1, 0, "clump", True), (300, 1, 3, "uniform", False),
    (300, 2, 1, "uniform", True), (300, 2, 1, "clump", False), (300, 1, 1, "uniform", False),
])
def test_same_grids_as_the_walk(n_grid, order, code, kind, weighted):
    torch = require_gpu()
    from paper_1512_07295_amd.estimator import Estimator

    box = 900.0
    rng = np.random.default_rng(n_grid + 10 * order + code)
    pos = rng.uniform(0, box, (50001, 3))
    if kind == "clump":  # past the 32-bit format
        pos[:9000] = np.mod(rng.normal(0.99 * box, 0.4 * box / n_grid, (9000, 3)), box)
    pos = pos.astype(np.float32)
    w = rng.exponential(1.0, len(pos)).astype(np.float32)
    grids = []
    for room in (len(pos), n_grid ** 3 // 4 + 1):
        est = Estimator(n_grid, box, order, code, 1, room, weighted=weighted)
        if weighted:
            est.set_weights(to_dev(torch, w))
        est.deposit(to_dev(torch, pos))
        grids.append([est.copy_grid(i + 1, 0) for i in range(2 ** code)])
        est.close()
    total = w.astype(np.float64).sum() if weighted else len(pos)
    for a, b in zip(*grids):
        # fixed-point sums of the same terms
        assert torch.equal(a, b)
        assert abs(float(a.double().sum()) - total) <= 1e-5 * total
