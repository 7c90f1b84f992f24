"""Transverse maps on planes whose tables hold fewer steps than a chunk of 64:
steps run in pairs up to the end of the tables; the fields are the same bits
wherever a call or a table ends, and the oracle's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.test_gpu_step_pairs import _calls, _wl  # noqa: E402
from tests.util import oracle_run, rel_l2  # noqa: E402


@pytest.mark.parametrize("shape,nf", [((192, 144, 2), 2), ((256, 256, 1), 3), ((144, 256, 8), 3)])
@pytest.mark.parametrize("order", [0, 1])
def test_calls_across_the_tables_give_the_same_bits(shape, nf, order):
    """41 steps: two or more fillings of the tables (27, 11 and 20 steps)."""
    wl = _wl(shape, nf, 41, "map", seed=sum(shape))
    whole, _, _ = _calls(wl, [41], order)
    parts, _, _ = _calls(wl, [1, 26, 3, 11], order)
    watched, _, _ = _calls(wl, [41], order, monitor=10)
    for a, b, c in zip(whole, parts, watched):
        assert torch.equal(a, b) and torch.equal(a, c)
    # about 3e-7 of rounding a step, growing with its square root
    for a, r in zip(whole, oracle_run(wl)):
        assert np.isfinite(a.cpu().numpy()).all()
        assert rel_l2(a.cpu().numpy(), r.numpy()) < 1e-5
