"""Calls whose steps the library takes by one-kernel steps or by the per-pass
kernels, as sizes, grid, sub-cycle, measuring and the steps of a run decide,
bit for bit against the per-pass kernels throughout (pic_set_pipeline off): a
discharge that always keeps the passes (one step-kernel workgroup per CU, ions
at rest on most steps: the pipelined electron passes through the default
dispatch), one that changes with the length of the call, and one that changes
when measuring starts. And batches, whose steps take one launch for all their
discharges or one per pass by the same kind of rule: unlike discharges (grids,
sub-cycles, sorts, variants, a species of odd tiles) beside each other, through
calls of which some take either."""
import numpy as np
import pytest

from gpu_common import need_gpu
from helpers import ANISO, NO_FIELD, OPAL, RECORD
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


# (electrons, ions), parameters of a batch's discharges
BATCH = [
    ((300_001, 299_999), dict(n_cells=4096, ion_subcycle=7, sort_interval=11)),
    ((2049, 2511), dict(n_cells=64, ion_subcycle=1, sort_interval=3)),
    ((260_003, 250_001), dict(n_cells=1500, ion_subcycle=10, sort_interval=0,
                              flags=RECORD | ANISO | OPAL)),
    ((0, 9001), dict(n_cells=2048, ion_subcycle=2, sort_interval=50, flags=RECORD | NO_FIELD)),
]


def test_batches_on_either_route_equal_passes():
    import torch

    from paper_2109_04469_amd import Batch

    s = torch.cuda.current_stream()
    ds, refs = [], []
    for n, over in BATCH:
        p, init = _setup(n, over)
        ds.append(_new(p, init, s))
        refs.append(_new(p, init))
        refs[-1].set_pipeline(False)
    batch = Batch(ds)
    # more than half a million particles on a grid that leaves a step kernel one
    # workgroup per CU: measuring, or with ions mostly at rest, the passes
    calls = ((1, ()), (70, ()), (5, (0, 2)), (1, (0, 2)), (2, (1,)), (66, (0, 1, 2, 3)), (3, ()))
    for k, (steps, measuring) in enumerate(calls):
        print(f"[route] batch: call {k} of {steps} steps", flush=True)
        for i, (d, r) in enumerate(zip(ds, refs)):
            for a in (d, r):
                a.measure(i in measuring)
            r.step(steps)
        batch.step(steps)
        if k == 3:
            ds[1].step(4)  # a discharge on its own between two calls of the batch
            refs[1].step(4)
        for i, (d, r) in enumerate(zip(ds, refs)):
            _same(d, r, f"batch, call {k}, discharge {i}")
    for d, r in zip(ds, refs):
        a, b = d.moments(), r.moments()
        assert a["steps"] == b["steps"]
        for key in ("n_e", "n_i", "eepf"):
            assert np.array_equal(a[key], b[key]), key
        np.testing.assert_allclose(a["mean_energy_e"], b["mean_energy_e"], rtol=1e-12)
    batch.close()
