"""GPU grids of the z-walking deposit (orders 1..4 on grids larger than a tile)
against the oracle at the sizes where its tiles, rounds and formats change."""

import numpy as np
import pytest

from gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu


def _sets(kind, box, n_grid, seed):
    """Particle sets of a batch: uniform, one dense clump, or a batch with an
    empty set between a sparse and a dense one."""
    rng = np.random.default_rng(seed)
    uniform = rng.uniform(0, box, (6000, 3))
    # about 4000 particles in a few cells: more than the 32-bit format allows
    # in one bucket, and several rounds of candidates in one tile
    clump = np.mod(rng.normal(0.97 * box, 0.4 * box / n_grid, (4000, 3)), box)
    if kind == "uniform":
        return [uniform]
    if kind == "clump":
        return [np.concatenate([uniform[:500], clump])]
    return [uniform[:40], uniform[:0], np.concatenate([uniform[:2000], clump[:600]])] * 8


# 20: the smallest walked grid (a ragged tile of 4 cells on every axis); 24, 40:
# ragged in x and y, whole in z; 32: whole tiles; 100: ragged in z too, and with 24
# sets more units than resident workgroups (units taken from the counter)
@pytest.mark.parametrize("n_grid,order,code,kind,weighted", [
    (20, 4, 1, "uniform", False), (20, 1, 0, "clump", False), (20, 3, 2, "uniform", True),
    (24, 3, 1, "clump", True), (24, 2, 3, "uniform", False), (32, 4, 1, "clump", False),
    (32, 2, 0, "clump", True), (40, 4, 2, "clump", True), (40, 1, 1, "uniform", True),
    (100, 4, 0, "uniform", False), (100, 2, 1, "clump", False),
    (100, 4, 1, "batch", False), (100, 3, 0, "batch", True),
])
def test_grids_against_the_oracle(n_grid, order, code, kind, weighted):
    torch = require_gpu()
    from oracle.assign import deposit_u, grid_coords
    from oracle.spectrum import mask_shift, shift_masks
    from paper_1512_07295_amd.estimator import Estimator

    box = 700.0
    sets = _sets(kind, box, n_grid, 1000 * n_grid + order)
    pos = np.concatenate(sets).astype(np.float64)
    w = np.random.default_rng(5).exponential(1.0, len(pos)).astype(np.float32) if weighted else None
    est = Estimator(n_grid, box, order, code, len(sets), len(pos), weighted=weighted)
    if weighted:
        est.set_weights(to_dev(torch, w))
    ends = np.cumsum([len(s) for s in sets])
    offs = None if len(sets) == 1 else to_dev(torch, np.concatenate([[0], ends]).astype(np.int64))
    est.deposit(to_dev(torch, pos), offs)
    for m, s in enumerate(sets):
        lo = ends[m] - len(s)
        ws = None if w is None else w[lo:ends[m]].astype(np.float64)
        for which, mask in enumerate(shift_masks(code)):
            got = est.copy_grid(which + 1, m).cpu().numpy()
            if len(s) == 0:
                assert not got.any()
                continue
            u = grid_coords(s, box, n_grid) + mask_shift(mask)[None, :]
            ref = deposit_u(u, order, n_grid, weights=ws)
            # float32 grids of float32 weights: 2e-6 of the largest value
            assert np.max(np.abs(got - ref)) <= 2e-6 * np.max(ref), (m, mask)
    est.close()
