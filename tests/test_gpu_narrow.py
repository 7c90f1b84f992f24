"""Passes with one field per thread (launches of few waves) and passes with
the fields together in a thread: shapes on both sides of the line between
them and at the edges of their blocks, against the oracle; and batches whose
groups take the one kernel while their problems alone take the other, bit for
bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2609_08384_amd import brahms, inputs  # noqa: E402
from tests.util import oracle_run, rel_l2  # noqa: E402

DEV = "cuda:0"


def _wl(shape, nf, nz, seed, dk=1.3):
    nx, ny, nt = shape
    fs = [inputs.FieldSpec(kappa=1.0 - 0.2 * j, diffraction=0.4 + 0.2 * j, tan_rho=0.3 * j, delay=0.5 - 0.4 * j,
                           k2=0.6 - 0.5 * j) for j in range(nf)]
    rng = np.random.default_rng(seed)
    wl = inputs.Workload("narrow", nx, ny, nt, nf, nz, 0.01, fs, dk_const=dk)
    wl.init = inputs.random_fields(rng, nf, nx, ny, nt, scale=0.7, smooth=max(1.0, min(shape) / 2.0))
    return wl


# x lines of length 16 take 4 lanes: 128 x 256 lines are 2048 waves of lanes
# (fields together), 96 x 256 are fewer; 3 and 5 leave partial blocks on every
# axis; 72, 36, 18, 24: values not a multiple of the field count per lane
@pytest.mark.parametrize("shape,nf", [((16, 128, 256), 2), ((16, 96, 256), 3), ((3, 6, 9), 3), ((8, 3, 12), 2),
                                      ((72, 36, 18), 3), ((24, 48, 4), 2), ((256, 9, 16), 3), ((64, 128, 192), 2)])
@pytest.mark.parametrize("merge,fuse", [(0, 0), (1, 1)])
def test_few_and_many_waves_match_oracle(shape, nf, merge, fuse):
    """Four steps: about 3e-7 of rounding per step on fields whose parts are
    all transformed and coupled, well below 1e-5; a wrong point, field or
    line gives O(1)."""
    wl = _wl(shape, nf, 4, 31 + nf)
    out = brahms.run_workload(wl, device=DEV, pass_order=(nf + shape[1]) % 4, merge_halves=merge, fuse_steps=fuse)
    for a, r in zip(out, oracle_run(wl, merge=bool(merge))):
        assert rel_l2(a.cpu().numpy(), r.numpy()) < 1e-5


@pytest.mark.parametrize("shape,nf,count", [((32, 48, 32), 2, 25), ((48, 36, 32), 3, 32), ((12, 64, 64), 2, 25)])
@pytest.mark.parametrize("merge", [0, 1])
def test_batch_groups_past_the_line_equal_plans(shape, nf, count, merge):
    """Problems that alone take the one-field-per-thread passes, in launch
    groups whose lines together take the others (and a last group of one)."""
    wls = [_wl(shape, nf, 3 + k % 4, 50 + k, dk=0.2 * k) for k in range(count)]
    fields = [[torch.from_numpy(a).to(DEV) for a in w.init] for w in wls]
    batch = brahms.Batch([(w.nx, w.ny, w.nt, w.nf, brahms.params_from_workload(w), w.nz) for w in wls])
    batch.set_merge_halves(merge)
    batch.set_fuse_steps(merge)
    batch.set_schedule(count - 1)
    batch.bind(fields)
    batch.run()
    torch.cuda.synchronize()
    for w, fs in zip(wls, fields):
        alone = brahms.run_workload(w, device=DEV, pass_order=0, merge_halves=merge, fuse_steps=merge)
        for a, b in zip(fs, alone):
            assert torch.equal(a, b), w.nz
    batch.destroy()
