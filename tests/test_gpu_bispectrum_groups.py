"""The bispectrum of every triangle, whose jobs take several groups of
workgroups, against the same triangles among a few, which take one."""

import numpy as np
import pytest

from oracle import bispectrum
from gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu


# two groups of 65 jobs; three; five; eight, the last one of 100 jobs
@pytest.mark.parametrize("n_grid,n_bins", [(180, 56), (256, 84), (320, 100), (400, 128)])
def test_few_triangles_of_many(n_grid, n_bins):
    torch = require_gpu()
    from paper_1512_07295_amd.estimator import Estimator

    box = 400.0
    rng = np.random.default_rng(n_bins)
    pos = rng.uniform(0, box, (200000, 3))
    pos = np.mod(pos + 0.05 * box * np.sin(2 * np.pi * pos[:, ::-1] / box), box)
    tri = bispectrum.closed_triangles(n_bins)
    some = np.sort(rng.choice(len(tri), 60, replace=False))
    est = Estimator(n_grid, box, 4, 1, 1, len(pos))
    est.power(to_dev(torch, pos))
    b, n_tri = (t.cpu().numpy()[some] for t in est.bispectrum(tri, 1, n_bins))
    few, n_few = (t.cpu().numpy() for t in est.bispectrum(np.asarray(tri)[some], 1, n_bins))
    # chunk sums are the same; float64 sums of 10^6 chunks in another order
    assert np.all(np.abs(n_tri - n_few) <= 1e-9 * n_few)
    assert np.all(np.abs(b - few) <= 1e-7 * np.abs(few) + 1e-9 * np.max(np.abs(few)))
    est.close()
