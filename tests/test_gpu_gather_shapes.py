"""Adjoint gather at the edges of its split: particle counts around the
particles of a wave and of a workgroup (one, two or four lanes per particle),
stencils that pass the end of every axis, packed and complex grids, both
position types.

dL/dx within 1e-4 of max |dL/dx| of the FP64 oracle gradient (the bound of
the other adjoint tests: FP32 grids and sums)."""

import numpy as np
import pytest

from oracle import adjoint
import synth
from gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("code,dtype,count", [(0, np.float32, 17), (0, np.float64, 257), (1, np.float32, 65),
                                              (1, np.float64, 15), (2, np.float32, 129), (3, np.float64, 63)])
def test_gradient_at_wave_edges(torch, p, code, dtype, count):
    from paper_1512_07295_amd.estimator import Estimator
    n, box = 24, 240.0
    pos = synth.uniform(count, box, 100 * p + count, dtype)
    # every third particle next to the end of an axis, on either side
    h = box / n
    edge = np.array([0.0, 0.3 * h, box - 0.3 * h, box - 1.2 * h, box - 1.7 * h, box - 2.4 * h])
    for i in range(0, count, 3):
        pos[i, (i // 3) % 3] = edge[(i // 9) % 6]
    pos[0] = box - 0.4 * h
    nb = n // 2
    dldp = np.linspace(1.0, 2.0, nb) / box ** 3
    est = Estimator(n, box, p, code, 1, count)
    gr = est.backward(to_dev(torch, pos), torch.tensor(dldp, device="cuda")).cpu().numpy()
    est.close()
    ref = adjoint.position_gradient(pos, box, n, p, code, 1, nb, dldp)
    assert np.max(np.abs(gr - ref)) <= 1e-4 * np.max(np.abs(ref))
