"""The one-kernel step (the default, and every batch) against the per-pass
kernels (pic_set_pipeline off), bit for bit:
states, decisions, counters, deposits and fields, at the edges of its tiles
(512 and 2048 slots), of the grids whose field its workgroups solve for
themselves, and with workgroups that take more tiles than a queue entry can
name without the queue being emptied. Both paths do the same FP64 operations
in the same order and sum integers, so the tolerance is zero; only the mean
energy, an FP64 sum in any order of at most a few million terms, is compared
at 1e-12."""
import numpy as np
import pytest

from gpu_common import assert_state_equal, near_wall_state, need_gpu
from helpers import ANISO, MAR, ME, OPAL, QE, RECORD, THOMAS
from pic_inputs import workloads, xsec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _setup(n, over):
    w = workloads.scaled(workloads.get("c1_small"), max(n), capacity_factor=3)
    p = dict(w["params"], reflection=0.3, gamma_see=0.3, pressure_pa=60.0, rf_voltage_v=200.0,
             flags=RECORD)
    p.update(over)
    dt = 1.0 / (p["rf_freq_hz"] * p["steps_per_cycle"])
    init = {}
    for sp, (T, m) in enumerate(((8.0, ME), (20.0, MAR))):
        v = np.sqrt(T * QE / m)
        k = 1 if sp == 0 else p["ion_subcycle"]
        init[sp] = near_wall_state(max(n[sp], 1), p["gap_m"], v, v * dt * k, 17, sp)
        init[sp] = tuple(a[:n[sp]] for a in init[sp])
    return p, init


def _new(p, init, stream=None):
    from paper_2109_04469_amd import Discharge

    d = Discharge(p, xsec.argon_synthetic(), stream=stream)
    for sp in (0, 1):
        d.set_state(sp, *init[sp], step=0)
    return d


def _same(a, b, what, record=True):
    assert a.sync() == 0 and b.sync() == 0, what
    for sp in (0, 1):
        assert_state_equal(a.get_state(sp), b.get_state(sp), what=f"{what} species {sp}")
        if record:
            assert np.array_equal(a.decisions(sp), b.decisions(sp)), f"{what}: decisions {sp}"
    assert np.array_equal(a.counters(), b.counters()), f"{what}: counters"
    fa, fb = a.get_field(), b.get_field()
    for k in ("rho", "phi", "E", "dep_e", "dep_i"):
        assert np.array_equal(fa[k], fb[k]), f"{what}: {k}"


EDGES = [
    # (electrons, ions), cells, ion sub-cycle, sort interval, flags, measure
    ((1, 0), 64, 1, 0, 0, False),
    ((511, 513), 2, 1, 4, 0, True),
    ((512, 512), 255, 2, 0, 0, False),
    ((2047, 2049), 256, 1, 5, 0, True),
    ((2048, 6001), 257, 3, 7, ANISO | OPAL, True),
    ((9001, 4097), 1024, 4, 0, 0, True),   # the largest grids solved by each workgroup,
    ((9001, 4097), 1025, 1, 6, 0, True),   # with few and with many nodes per thread
    ((3001, 8190), 2048, 2, 5, 0, True),
    ((3001, 8190), 2049, 5, 0, 0, True),   # a field launch before the step
    ((5003, 5003), 100, 1, 0, THOMAS, False),
]


@pytest.mark.parametrize("case", EDGES, ids=[f"{c[0][0]}-{c[1]}-{c[2]}" for c in EDGES])
def test_step_kernel_equals_per_pass_kernels(case):
    import torch

    from paper_2109_04469_amd import Batch

    n, cells, sub, sort, flags, measure = case
    p, init = _setup(n, dict(n_cells=cells, ion_subcycle=sub, sort_interval=sort,
                             flags=RECORD | flags))
    s = torch.cuda.current_stream()
    one, off, many, other = _new(p, init), _new(p, init), _new(p, init, s), _new(p, init, s)
    off.set_pipeline(False)
    batch = Batch([other, many])
    for d in (one, off, many):
        d.measure(measure)
    for k, steps in enumerate((1, 2, 19)):
        print(f"[step] {n} cells {cells}: call {k} of {steps} steps", flush=True)
        one.step(steps)
        off.step(steps)
        batch.step(steps)
        _same(one, off, f"call {k}")
        _same(many, off, f"batch, call {k}")
    if measure:
        mo = off.moments()
        for d in (one, many):
            m = d.moments()
            for key in ("n_e", "n_i", "eepf"):
                assert np.array_equal(m[key], mo[key]), key
            np.testing.assert_allclose(m["mean_energy_e"], mo["mean_energy_e"], rtol=1e-12)
            w, wo = d.wall_moments(), off.wall_moments()
            assert np.array_equal(w["arrivals"], wo["arrivals"])
            assert np.array_equal(w["fedf"], wo["fedf"])
    batch.close()


@pytest.mark.parametrize("n", [1_040_001, 4_700_001])
def test_step_kernel_with_long_runs_of_tiles(n):
    # one workgroup per CU: 16 small tiles each (1.04M + 1.04M particles), or
    # 17 large ones (4.7M + 4.7M)
    p, init = _setup((n, n), dict(n_cells=900, sort_interval=3, ion_subcycle=1, flags=0))
    one, off = _new(p, init), _new(p, init)
    off.set_pipeline(False)
    one.set_launch(1, 1)
    for steps in (1, 4):
        one.step(steps)
        off.step(steps)
        _same(one, off, f"{n} after {steps}", record=False)


def test_step_kernel_and_passes_in_turn():
    # one discharge whose calls alternate between the step kernel, the
    # per-pass kernels and the pipelined passes (event timers on): every
    # path starts from what the others leave
    p, init = _setup((6001, 5003), dict(n_cells=100, ion_subcycle=3, sort_interval=9))
    one, off = _new(p, init), _new(p, init)
    off.set_pipeline(False)
    for k, steps in enumerate((4, 1, 7, 5, 2, 11)):
        one.set_pipeline(k % 3 != 1)
        one.timing(1 if k % 3 == 2 else 0)
        one.step(steps)
        off.step(steps)
        _same(one, off, f"call {k}")
