"""The reverse sweep's paired passes (the end of one step and the beginning of
the next in one pass, inside a segment) against the same sweep with a segment
per step, which has none.

Both sweeps do the same products in another axis order: per pass the FP32
transforms add about 3e-7 of relative error, and 2 x 3 passes over 5 steps in
quadrature give 1.6e-6; the bound is six times that.  The dk gradient sums
terms of both signs over the grid, a factor of ten more.
"""
import numpy as np
import pytest

from tests.test_gpu_adjoint import _case, _gpu_grads
from tests.util import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("shape,nf", [((128, 4, 64), 2), ((96, 3, 48), 3), ((256, 2, 16), 2), ((9, 6, 192), 2),
                                      ((3, 9, 18), 3), ((72, 2, 256), 3), ((1, 6, 32), 2), ((64, 1, 1), 2)])
def test_paired_sweep_equals_single_steps(shape, nf, order):
    wl = _case(nf, shape, 5, seed=nf + sum(shape))
    j1, g1, d1, _ = _gpu_grads(wl, 1, order)
    j5, g5, d5, _ = _gpu_grads(wl, 5, order)
    assert abs(j1 - j5) <= 1e-6 * abs(j1)
    for a, b in zip(g1, g5):
        assert np.isfinite(b).all()
        assert rel_l2(b, a) < 1e-5
    assert rel_l2(d5, d1) < 1e-4
