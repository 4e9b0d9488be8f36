"""The general kernel's deposit of orders 1..4 on sparse grids: a batch of
equal sets, sparse enough for it, against one such set, which walks."""

import numpy as np
import pytest

from gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu


# 64: whole tiles; 72: ragged ones.  Batches of more cells than a 293^3 grid.
@pytest.mark.parametrize("n_grid,batch", [(64, 100), (72, 70)])
@pytest.mark.parametrize("code", [0, 1, 3])
@pytest.mark.parametrize("order,weighted", [(1, False), (2, True), (3, False), (3, True), (4, False), (4, True)])
def test_same_grids_as_the_walk(n_grid, batch, code, order, weighted):
    torch = require_gpu()
    from paper_1512_07295_amd.estimator import Estimator

    box, n = 300.0, 3001
    rng = np.random.default_rng(order + 10 * code)
    one = rng.uniform(0, box, (n, 3))
    one[:200] = np.mod(rng.normal(0, 2.0 * box / n_grid, (200, 3)), box)  # across the edges
    mass = rng.exponential(1.0, n).astype(np.float32)
    grids = []
    for b in (1, batch):
        est = Estimator(n_grid, box, order, code, b, b * n, weighted=weighted)
        if weighted:
            est.set_weights(to_dev(torch, np.tile(mass, b)))
        est.deposit(to_dev(torch, np.tile(one, (b, 1))), None if b == 1 else to_dev(torch, np.arange(b + 1) * np.int64(n)))
        grids.append([[est.copy_grid(i + 1, m) for i in range(2 ** code)] for m in sorted({0, b // 2, b - 1})])
        est.close()
    for member in grids[1]:
        for a, b in zip(grids[0][0], member):
            assert torch.equal(a, b)  # fixed-point sums of the same terms
