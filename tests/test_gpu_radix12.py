"""Run-time FFT lines with radix 12 in the middle (576 = 16 x 12 x 3, 960 = 16 x
12 x 5) and at the end (192 = 16 x 12): modes, P(k) and the gradient."""

import numpy as np
import pytest

import oracle
from oracle import adjoint
from gpu_common import rel_err, require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("code", [0, 1])
def test_192_power_and_gradient(code):
    torch = require_gpu()
    from paper_1512_07295_amd.estimator import Estimator

    n_grid, box, order, n_bins = 192, 600.0, 3, 96
    pos = np.random.default_rng(3).uniform(0, box, (3000, 3))
    est = Estimator(n_grid, box, order, code, 1, len(pos))
    x = to_dev(torch, pos)
    _, p, modes = est.power(x, n_bins=n_bins)
    _, p0, n0 = oracle.power(pos, box, n_grid, order, bool(code), 1, n_bins)
    assert np.array_equal(modes.cpu().numpy()[0], n0)
    assert rel_err(p.cpu().numpy()[0], p0) < 1e-5  # float32 grids
    dldp = np.cos(np.arange(n_bins))
    g = est.backward(x, to_dev(torch, dldp[None, :]), n_bins=n_bins).cpu().numpy()
    g0 = adjoint.position_gradient(pos, box, n_grid, order, bool(code), 1, n_bins, dldp)
    assert np.max(np.abs(g - g0)) < 1e-4 * np.max(np.abs(g0))
    est.close()


# rows of 192 (384 packed), 576 and 960
@pytest.mark.parametrize("n_grid,code", [(384, 0), (576, 1), (960, 1)])
def test_modes_of_the_deposited_grids(n_grid, code):
    """The exported modes and P(k) from float64 transforms of the same grids."""
    torch = require_gpu()
    from paper_1512_07295_amd.estimator import Estimator

    box, n, order = 500.0, 20000, 2
    pos = to_dev(torch, np.random.default_rng(n_grid).uniform(0, box, (n, 3)).astype(np.float32))
    est = Estimator(n_grid, box, order, code, 1, n)
    est.deposit(pos)
    m = torch.fft.fftfreq(n_grid, 1.0 / n_grid, device="cuda", dtype=torch.float64)
    m[n_grid // 2] = n_grid // 2
    mz = m[:n_grid // 2 + 1]
    c = None
    for which in range(2 ** code):
        f = torch.fft.rfftn(est.copy_grid(which + 1).double())
        if which:
            for x in range(n_grid):
                f[x] *= torch.exp(1j * np.pi / n_grid * (m[x] + m[:, None] + mz[None, :]))
        c = f if c is None else c.add_(f).mul_(0.5)
        del f
    est.transform()
    _, p, _ = est.power_only()
    d = est.export_delta()
    w = torch.sinc(m / n_grid) ** order
    worst = top = 0.0
    for x in range(n_grid):  # window times delta: rounding is relative to the field
        ref = c[x] / n
        got = torch.view_as_complex(d[x]) * (w[x] * w[:, None] * w[None, :n_grid // 2 + 1])
        worst, top = max(worst, float((got - ref).abs().max())), max(top, float(ref.abs().max()) if x else 1.0)
    assert worst < 1e-6 * top  # float32 transforms of up to 960 points per axis
    del c
    _, p0, _ = est.spectrum_power(d)
    assert rel_err(p.cpu().numpy()[0], p0.cpu().numpy()) < 1e-5
    est.close()
