"""The one-kernel step on its 2048-slot tiles (more than 4096 particles of both
species per compute unit), measuring or not, with and without the method
variants, alone and in a batch beside a small plain one, bit for bit against
the per-pass kernels."""
import numpy as np
import pytest

from gpu_common import need_gpu
from helpers import ANISO, OPAL, RECORD
from test_gpu_step_kernel import _new, _same, _setup

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("flags", [0, ANISO | OPAL], ids=["plain", "variants"])
@pytest.mark.parametrize("measure", [False, True], ids=["", "measuring"])
def test_large_tiles_equal_per_pass_kernels(flags, measure):
    import torch

    from paper_2109_04469_amd import Batch

    p, init = _setup((561_003, 560_001), dict(n_cells=300, ion_subcycle=2, sort_interval=5,
                                              flags=RECORD | flags))
    q, init2 = _setup((3001, 2049), dict(n_cells=64, flags=RECORD))
    s = torch.cuda.current_stream()
    one, off, many = _new(p, init), _new(p, init), _new(p, init, s)
    other, other_off = _new(q, init2, s), _new(q, init2)
    for d in (off, other_off):
        d.set_pipeline(False)
    batch = Batch([other, many])
    for d in (one, off, many):
        d.measure(measure)
    for steps in (1, 2, 9):
        print(f"[large] flags {flags} measure {measure}: call of {steps} steps", flush=True)
        one.step(steps)
        off.step(steps)
        other_off.step(steps)
        batch.step(steps)
        _same(one, off, f"after {steps}")
        _same(many, off, f"batch, after {steps}")
        _same(other, other_off, f"batch, the plain one, after {steps}")
    if measure:
        mo, wo = off.moments(), off.wall_moments()
        for d in (one, many):
            m, w = d.moments(), d.wall_moments()
            for key in ("n_e", "n_i", "eepf"):
                assert np.array_equal(m[key], mo[key]), key
            np.testing.assert_allclose(m["mean_energy_e"], mo["mean_energy_e"], rtol=1e-12)
            assert np.array_equal(w["arrivals"], wo["arrivals"])
            assert np.array_equal(w["fedf"], wo["fedf"])
    batch.close()
