"""The block -> tile map of the x and y passes (an eighth of the tiles in a row
for each XCD, the remainder as it comes): tile counts below, at and beside
multiples of eight, on lone plans and in batches, against the oracle.  A tile
left out or taken twice gives O(1); the bound is that of a few steps of FP32
rounding (3e-7 each), as for the narrow launches."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2609_08384_amd import brahms  # noqa: E402
from tests.test_gpu_narrow import DEV, _wl  # noqa: E402
from tests.util import oracle_run, rel_l2  # noqa: E402

# (x tiles, y tiles) of the one-field-per-thread kernels: lines of 4, 8 and 16
# lanes on x are 16, 8 and 4 to a tile
SHAPES = [((16, 6, 18), 2), ((16, 8, 16), 3), ((16, 9, 16), 2), ((48, 9, 48), 2), ((256, 6, 9), 2), ((64, 8, 9), 3),
          ((64, 256, 36), 2)]


@pytest.mark.parametrize("shape,nf", SHAPES)
@pytest.mark.parametrize("merge", [0, 1])
def test_every_tile_is_taken_once(shape, nf, merge):
    wl = _wl(shape, nf, 3, 7 + nf)
    ref = [r.numpy() for r in oracle_run(wl, merge=bool(merge))]
    for order in (0, 3):
        out = brahms.run_workload(wl, device=DEV, pass_order=order, merge_halves=merge, fuse_steps=merge)
        for a, r in zip(out, ref):
            assert rel_l2(a.cpu().numpy(), r) < 1e-5
    fields = [[torch.from_numpy(a).to(DEV) for a in wl.init] for _ in range(3)]
    batch = brahms.Batch([(wl.nx, wl.ny, wl.nt, nf, brahms.params_from_workload(wl), wl.nz)] * 3)
    batch.set_merge_halves(merge)
    batch.set_fuse_steps(merge)
    batch.bind(fields)
    batch.run()
    torch.cuda.synchronize()
    for fs in fields:
        for a, r in zip(fs, ref):
            assert rel_l2(a.cpu().numpy(), r) < 1e-5
    batch.destroy()
