"""GPU bispectrum against the oracle at the shapes where its launch changes:
planes per slab, jobs per wave, the second call that reuses the count sums.
Tolerances: N_tri to 1e-5 relative, B to 1e-5 of the larger of |B| and
V^2 sum|III| / sum JJJ (B can cross zero)."""

import numpy as np
import pytest

import oracle
from oracle import bispectrum, spectrum
from gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu


# (N, n_dk, n_bins): one shell; five (at most one job per wave); twelve; twenty
# (more jobs than waves); wide shells
@pytest.mark.parametrize("n_grid,n_dk,n_bins", [(16, 1, 1), (24, 1, 5), (48, 1, 12), (72, 1, 20), (60, 3, 5)])
def test_bispectrum_of_every_triangle(n_grid, n_dk, n_bins):
    torch = require_gpu()
    from paper_1512_07295_amd.estimator import Estimator

    box = 400.0
    pos = np.random.default_rng(n_grid + n_bins).uniform(0, box, (4000, 3))
    pos = np.mod(pos + 0.1 * box * np.sin(2 * np.pi * pos[:, ::-1] / box), box)
    tri = bispectrum.closed_triangles(n_bins)
    _, b0, n0 = oracle.bispectrum_fn(pos, box, n_grid, 4, True, n_dk=n_dk, n_bins=n_bins, triangles=tri)
    delta, _ = spectrum.delta_half(pos, box, n_grid, 4, True)
    masks = bispectrum.shell_masks(n_grid, n_dk, n_bins)
    s_abs = bispectrum.triple_sums(np.abs(bispectrum.shell_fields(delta, masks, n_grid)), tri)
    s_jjj = bispectrum.triple_sums(bispectrum.shell_fields(np.ones_like(delta), masks, n_grid), tri)
    scale = np.maximum(np.abs(b0), box ** 6 * s_abs / s_jjj)
    est = Estimator(n_grid, box, 4, 1, 1, len(pos))
    est.power(to_dev(torch, pos))
    for _ in range(2):
        b, n_tri = est.bispectrum(tri, n_dk, n_bins)
        ok = n0 > 0.5
        assert np.all(np.abs(n_tri.cpu().numpy() - n0) <= 1e-5 * n0 + 1e-3)
        assert np.all(np.abs(b.cpu().numpy() - b0)[ok] <= 1e-5 * scale[ok])
    est.close()
