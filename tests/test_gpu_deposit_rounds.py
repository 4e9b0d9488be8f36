"""The z-walking deposit of one grid at the particle counts of one tile where
its rounds of 512 and 1024 candidates begin and end."""

import numpy as np
import pytest

from gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu

WIDE = 33  # launch choice: the defaults with the 64-bit format


@pytest.mark.parametrize("order", [1, 2, 3, 4])
@pytest.mark.parametrize("weighted", [False, True])
def test_candidates_of_one_tile(order, weighted):
    torch = require_gpu()
    from oracle.assign import deposit_u, grid_coords
    from paper_1512_07295_amd.estimator import Estimator

    n_grid, box = 40, 40.0
    rng = np.random.default_rng(order)
    est = Estimator(n_grid, box, order, 0, 1, 5000, weighted=weighted)
    for n in (1, 63, 511, 512, 513, 1023, 1024, 1025, 1537, 2048, 2049):
        # stencils inside the tile of cells 16..31 in x and y, 8..15 in z
        pos = rng.uniform((18, 18, 10), (30, 30, 14), (n, 3))
        w = rng.exponential(1.0, n).astype(np.float32) if weighted else None
        if weighted:
            est.set_weights(to_dev(torch, w))
        ref = deposit_u(grid_coords(pos, box, n_grid), order, n_grid, weights=None if w is None else w.astype(float))
        for choice in (35, WIDE):  # 35: the defaults
            est.set_launch(choice)
            est.deposit(to_dev(torch, pos))
            got = est.copy_grid().cpu().numpy()
            assert np.max(np.abs(got - ref)) <= 2e-6 * np.max(ref), (n, choice)  # float32 grid and weights
    est.close()
