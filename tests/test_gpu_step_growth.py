"""A discharge that grows far beyond what the host last saw within one call of
pic_step keeps the 512-slot tiles it started with: its workgroups then take
more tiles than a queue entry can name (16) and more than a workgroup sums in
LDS (64 output tiles). Hot electrons in a dense gas double every two steps; one
workgroup per CU ends the call with more than a hundred tiles each. Bit for bit
against the per-pass kernels. Afterwards, and through long calls that nobody
reads in between, the counts that arrive by themselves may change the tiles and
the route from one sort to the next: the same bits again."""
import numpy as np
import pytest

from gpu_common import need_gpu
from helpers import MAR, ME, NO_FIELD, QE
from pic_inputs import workloads
from test_gpu_step_kernel import _new, _same, _setup

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def test_one_call_that_outgrows_its_tiles():
    n = 200_000
    w = workloads.scaled(workloads.get("c1_small"), n, capacity_factor=60)
    p = dict(w["params"], pressure_pa=3000.0, flags=NO_FIELD, sort_interval=0, ion_subcycle=1,
             reflection=0.5, gamma_see=0.0)
    rng = np.random.default_rng(1)
    init = {}
    for sp, (ev, m) in enumerate(((2000.0, ME), (0.03, MAR))):
        v = rng.normal(size=(3, n))
        v *= np.sqrt(2.0 * ev * QE / m / (v**2).sum(axis=0))
        init[sp] = (rng.uniform(0.1, 0.9, n) * p["gap_m"], *(np.ascontiguousarray(c) for c in v))
    one, off = _new(p, init), _new(p, init)
    off.set_pipeline(False)
    one.set_launch(1, 1)
    for steps in (16, 2):
        one.step(steps)
        off.step(steps)
        _same(one, off, f"after {steps} more", record=False)
        assert one.count(0) + one.count(1) > 65 * 512 * 256


@pytest.mark.parametrize("sort", [0, 50, 300])
def test_long_calls_that_nobody_reads(sort):
    p, init = _setup((9001, 8003), dict(n_cells=100, sort_interval=sort, flags=0))
    one, off = _new(p, init), _new(p, init)
    off.set_pipeline(False)
    for steps in (700, 3, 260, 511):
        one.step(steps)
        off.step(steps)
    _same(one, off, "at the end", record=False)
