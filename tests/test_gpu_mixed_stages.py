"""P(k), sampled modes and the adjoint on grids whose FFT plans use every
stage of the run-time lines: first radices 16, 12, 10, 8, 6, 4, 2, grouped
radices 6, 9, 10, 12, 15 in the middle and at the end."""

import numpy as np
import pytest

import oracle
from oracle import adjoint, spectrum
from gpu_common import rel_err, require_gpu, to_dev

pytestmark = pytest.mark.gpu


# N (one grid: rows of N/2): 20 (rows 10), 24 (8 x 3; 12), 36 (12 x 3; 18 = 6 x 3), 60 (12 x 5;
# 30 = 6 x 5), 72 (8 x 9), 96 (16 x 6), 120 (8 x 15), 144 (16 x 9), 160 (16 x 10)
@pytest.mark.parametrize("n_grid", [20, 24, 36, 60, 72, 96, 120, 144, 160])
@pytest.mark.parametrize("code", [0, 1])
def test_power_modes_and_gradient(n_grid, code):
    torch = require_gpu()
    from paper_1512_07295_amd.estimator import Estimator

    box, order, n_bins = 600.0, 3, n_grid // 2
    pos = np.random.default_rng(n_grid).uniform(0, box, (3000, 3))
    est = Estimator(n_grid, box, order, code, 1, len(pos))
    x = to_dev(torch, pos)
    _, p, modes = est.power(x, n_bins=n_bins)
    _, p0, n0 = oracle.power(pos, box, n_grid, order, bool(code), 1, n_bins)
    assert np.array_equal(modes.cpu().numpy()[0], n0)
    assert rel_err(p.cpu().numpy()[0], p0) < 1e-5  # float32 grids
    delta, _ = spectrum.delta_half(pos, box, n_grid, order, bool(code))
    m = np.random.default_rng(1).integers(-(n_grid // 2) + 1, n_grid // 2, (200, 3))
    m[:, 2] = np.abs(m[:, 2])
    got = est.sample_delta(m).cpu().numpy()
    ref = delta[m[:, 0] % n_grid, m[:, 1] % n_grid, m[:, 2]]
    # rounding is relative to the field, and the window divides it: compare with the window on
    w = spectrum.window_1d(order, m, n_grid).prod(axis=1)
    assert np.max(np.abs(got - ref) * w) < 1e-5 * np.max(np.abs(ref) * w)
    if n_grid <= 96:
        dldp = np.cos(np.arange(n_bins))
        g = est.backward(x, to_dev(torch, dldp[None, :]), n_bins=n_bins).cpu().numpy()
        g0 = adjoint.position_gradient(pos, box, n_grid, order, bool(code), 1, n_bins, dldp)
        assert np.max(np.abs(g - g0)) < 1e-4 * np.max(np.abs(g0))
    est.close()
