"""The reverse sweep with the three fields together in a thread (launches that
fill the chip), against the oracle's adjoint: the smallest launches on that
side of the line, x and tau lines of 8 and 16 lanes, segments of one step and
of two.  Bounds as for the other sweeps (test_gpu_adjoint.py): two steps add
less rounding than the twelve there."""
import numpy as np
import pytest

from tests.test_gpu_adjoint import _case, _gpu_grads, _oracle_grads
from tests.util import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(128, 128, 128), (256, 128, 64)])
def test_three_fields_together_match_oracle(shape):
    wl = _case(3, shape, 2, seed=sum(shape))
    jo, go, gdko = _oracle_grads(wl)
    for order, every in ((0, 2), (1, 1)):
        jg, g, gdk, _ = _gpu_grads(wl, every, order)
        assert abs(jg - jo) < 1e-5 * abs(jo)
        for j in range(3):
            assert np.isfinite(g[j]).all()
            assert rel_l2(g[j], go[j]) < 1e-4, (order, j)
        assert rel_l2(gdk, gdko) < 1e-4, order
