"""Further call sequences on the host emulation (see test_host_emulation.py):
literal steps in pairs with a transverse map, maps whose tables hold a few
steps, graph replays of chunks that begin with an even and with an odd
step (plane waves, two axes, three axes, literal and merged), the x and y
passes that take their tiles in slabs, and the adjoint.
Plane-wave launches are checked row by row over all the steps they take, and
adjoint passes over their states, tables and partial sums."""
import os
import subprocess

import pytest

from tests import test_host_emulation as emu


@pytest.fixture(scope="module")
def drive():
    if emu._clang() is None:
        pytest.skip("clang++ not available")
    out = os.path.join(emu.EMU, "_build", emu._source_hash())
    exe = os.path.join(out, "drive")
    if not os.path.exists(exe):
        exe = emu._build(out)["drive"]
    return exe


@pytest.mark.parametrize("scenario", ["maps", "large_map", "slabs", "graph_chunks", "adjoint"])
def test_scenario_under_sanitizers(drive, scenario):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0:abort_on_error=1",
               UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
    emu._check(subprocess.run([drive, scenario], capture_output=True, text=True, env=env, timeout=1800))
