"""Mass sums whose partial results share memory with a later pass: P(k) of one
set after another on one handle, and the direct sum with masses in its least
workspace."""

import numpy as np
import pytest

import oracle
from oracle import direct
from gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu


# 8 with one set: the fewest partial sums beside 1024 slices; 40 sets: 51 slices each
@pytest.mark.parametrize("n_grid,batch", [(8, 1), (16, 3), (24, 40)])
def test_masses_change_between_calls(n_grid, batch):
    torch = require_gpu()
    from paper_1512_07295_amd.estimator import Estimator

    box, rng, n_bins = 100.0, np.random.default_rng(n_grid), n_grid // 2
    est = Estimator(n_grid, box, 2, True, batch, 3000, weighted=True)
    for n in (3000, 257, batch):
        cuts = np.linspace(0, n, batch + 1).astype(np.int64)
        pos, w = rng.uniform(0, box, (n, 3)), rng.exponential(1.0, n).astype(np.float32)
        est.set_weights(to_dev(torch, w))
        _, p, _ = est.power(to_dev(torch, pos), to_dev(torch, cuts) if batch > 1 else None, subtract_shot=True)
        p = p.cpu().numpy()
        for m in sorted({0, batch // 2, batch - 1}):
            s = slice(cuts[m], cuts[m + 1])
            _, ref, _ = oracle.power(pos[s], box, n_grid, 2, True, 1, n_bins, subtract_shot=True, weights=w[s])
            shot = box ** 3 * np.sum(w[s].astype(float) ** 2) / np.sum(w[s].astype(float)) ** 2
            assert np.max(np.abs(p[m] - ref)) < 1e-5 * (np.max(np.abs(ref)) + shot)  # float32 grids
    # an invalid mass anywhere makes the call's results NaN, and only that call's
    for bad in (np.nan, np.inf, -1.0):
        v = w.copy()
        v[-1] = bad
        est.set_weights(to_dev(torch, v))
        assert torch.isnan(est.power(to_dev(torch, pos), to_dev(torch, cuts) if batch > 1 else None)[1]).all()
    est.set_weights(to_dev(torch, w))
    assert torch.isfinite(est.power(to_dev(torch, pos), to_dev(torch, cuts) if batch > 1 else None)[1]).all()
    est.close()


@pytest.mark.parametrize("n_grid,n", [(8, 1), (8, 2500), (12, 700)])
def test_direct_sum(n_grid, n):
    torch = require_gpu()
    import paper_1512_07295_amd as lib
    from paper_1512_07295_amd.estimator import Estimator

    box, rng = 100.0, np.random.default_rng(n)
    pos, w = rng.uniform(0, box, (n, 3)), rng.exponential(1.0, n).astype(np.float32)
    est = Estimator(n_grid, box, 2, True, 1, n, weighted=True)
    est.set_weights(to_dev(torch, w))
    x = to_dev(torch, pos)
    got = est.direct_delta(x)
    static = torch.empty_like(got)
    lib.estimator_direct_delta_noalloc(est.h, x, lib.EST_F64, n, static)
    est.stream.synchronize()
    assert torch.equal(got, static)
    ref = direct.delta_half_direct(pos, box, n_grid, weights=w)
    got = got.cpu().numpy()
    assert np.max(np.abs(got[..., 0] + 1j * got[..., 1] - ref)) < 1e-5  # FP32 phases and chunk sums, |delta| <= 1
    est.close()
