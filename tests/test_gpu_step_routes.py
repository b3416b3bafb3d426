"""Calls whose steps the library takes by one-kernel steps or by the per-pass
kernels, as sizes, grid, sub-cycle, measuring and the steps of a run decide,
bit for bit against the per-pass kernels throughout (pic_set_pipeline off): a
discharge that always keeps the passes (one step-kernel workgroup per CU, ions
at rest on most steps: the pipelined electron passes through the default
dispatch), one that changes with the length of the call, and one that changes
when measuring starts."""
import pytest

from gpu_common import need_gpu
from helpers import ANISO, OPAL, RECORD
from test_gpu_step_kernel import _new, _same, _setup

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


CASES = {
    # (electrons, ions), parameters, ((steps, measuring), ...)
    "passes": ((531_001, 530_003), dict(n_cells=4096, ion_subcycle=7, sort_interval=11),
               ((1, False), (5, False), (13, False), (12, True), (2, True), (9, False))),
    "passes with variants": ((531_001, 530_003), dict(n_cells=4096, ion_subcycle=6, sort_interval=0,
                                                      flags=RECORD | ANISO | OPAL),
                             ((7, False), (8, False))),
    "length of the call": ((1_600_001, 1_600_000), dict(n_cells=300, ion_subcycle=10, sort_interval=17),
                           ((1, False), (9, False), (1, False), (1, False), (13, False))),
    "measuring": ((800_001, 800_000), dict(n_cells=3000, ion_subcycle=2, sort_interval=50),
                  ((4, False), (4, True), (4, False), (5, True), (3, False))),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_calls_on_either_route_equal_passes(name):
    n, over, calls = CASES[name]
    p, init = _setup(n, over)
    one, off = _new(p, init), _new(p, init)
    off.set_pipeline(False)
    for k, (steps, measure) in enumerate(calls):
        print(f"[route] {name}: call {k} of {steps} steps", flush=True)
        for d in (one, off):
            d.measure(measure)
            d.step(steps)
        _same(one, off, f"{name}, call {k}")
