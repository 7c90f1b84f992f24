"""Whole 64-step chunks replayed from a plan's graphs, from even and from odd
steps, against launch-by-launch stepping, bit for bit: plane waves (a chunk in
one launch), two axes and three, literal and merged, with replays of one graph
before and after those of the other."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2609_08384_amd import brahms  # noqa: E402
from tests.test_gpu_narrow import DEV, _wl  # noqa: E402

CALLS = [3, 64, 130, 1, 64, 128, 67, 64]


def _run(wl, graph, merge):
    fields = [torch.from_numpy(a).to(DEV) for a in wl.init]
    plan = brahms.Plan(wl.nx, wl.ny, wl.nt, wl.nf, brahms.params_from_workload(wl))
    plan.set_schedule(0, graph, merge)
    plan.bind(fields)
    at = []
    for n in CALLS:
        plan.step(n)
        at.append([f.clone() for f in fields])
        torch.cuda.synchronize()
    plan.destroy()
    return at


@pytest.mark.parametrize("shape,nf", [((1, 1, 64), 2), ((1, 1, 36), 3), ((16, 12, 1), 2), ((8, 6, 12), 3)])
@pytest.mark.parametrize("merge", [0, 1])
def test_replayed_chunks_equal_launches(shape, nf, merge):
    wl = _wl(shape, nf, 4, 11 + nf)
    wl.dz = 1e-3
    for n, a, b in zip(CALLS, _run(wl, 0, merge), _run(wl, 1, merge)):
        for x, y in zip(a, b):
            assert torch.isfinite(torch.view_as_real(x)).all()
            assert torch.equal(x, y), n
