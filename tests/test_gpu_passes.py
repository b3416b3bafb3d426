"""The per-pass kernels where a call takes them: with event timers on, a call of
several steps runs the pipelined electron passes (the emit of a step decides
the next one), with the pipeline off separate decide and emit kernels compiled
for 512 or 256 threads. The states, grids and options that the pipeline's own
tests name, now that calls without timers take one kernel per step: variants,
the Thomas solver, the largest grid, an empty species, the smaller decide
workgroups, tiles beyond one per workgroup, capacity overflow. All bit for bit
against single unpipelined steps. And states that are not finite, on every
path: the error is latched, and the discharge usable again after set_state."""
import numpy as np
import pytest

from gpu_common import near_wall_state, need_gpu
from helpers import MAR, ME, RECORD
from pic_inputs import state, workloads, xsec
from test_gpu_pipeline import CASES, _pair, _same, _vth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _passes(p, init, block=512):
    """Pipelined passes (timers on) with that decide size, and the reference."""
    many, ref = _pair(p, xsec.argon_synthetic(), init)
    many.timing(1)
    many.set_decide_block(block)
    ref.set_pipeline(False)
    return many, ref


def _compare(many, ref, calls, what):
    for n in calls:
        print(f"[passes] {what}: call of {n} steps", flush=True)
        many.step(n)
        for _ in range(n):
            ref.step(1)
        _same(many, ref, f"{what}, call of {n}")


def _near_wall(w, p, seed):
    dt = 1.0 / (p["rf_freq_hz"] * p["steps_per_cycle"])
    ve, vi = _vth(8.0, ME), _vth(20.0, MAR)
    return {0: near_wall_state(w["n_init"][0], p["gap_m"], ve, ve * dt, seed, 0),
            1: near_wall_state(w["n_init"][1], p["gap_m"], vi, vi * dt * p["ion_subcycle"], seed, 1)}


@pytest.mark.parametrize("block", [512, 256])
@pytest.mark.parametrize("name", sorted(CASES))
def test_pipelined_passes_equal_single_steps(name, block):
    c = CASES[name]
    w = workloads.scaled(workloads.get(c["base"]), c["n"])
    # ions at rest on some steps, so that steps are pipelined at all
    p = dict(w["params"], **c["over"])
    p["ion_subcycle"] = max(p["ion_subcycle"], 3)
    many, ref = _passes(p, _near_wall(w, p, 3), block)
    _compare(many, ref, (1, 2, 37, 60), name)


@pytest.mark.parametrize("empty", [0, 1])
def test_pipelined_passes_from_an_empty_species(empty):
    w = workloads.scaled(workloads.get("c1_small"), 6000, capacity_factor=8)
    p = dict(w["params"], reflection=0.2, gamma_see=0.4, ion_subcycle=3, sort_interval=0,
             pressure_pa=20.0, rf_voltage_v=150.0, flags=RECORD)
    init = _near_wall(w, p, 5)
    init[empty] = (np.zeros(0),) * 4
    many, ref = _passes(p, init)
    _compare(many, ref, (1, 7, 22), f"empty species {empty}")
    assert many.count(empty) > 0


@pytest.mark.parametrize("block", [512, 256])
def test_passes_with_several_tiles_per_workgroup(block):
    w = workloads.scaled(workloads.get("c1_small"), 700_001)
    p = dict(w["params"], flags=RECORD, reflection=0.3, gamma_see=0.2, ion_subcycle=3)
    init = state.initial_state(w, seed=33)
    many, ref = _passes(p, init, block)
    off, _ = _pair(p, xsec.argon_synthetic(), init)
    off.set_pipeline(False)
    off.set_decide_block(block)
    for d in (many, off):
        d.set_launch(1, 1)
    for n in (1, 5):
        many.step(n)
        off.step(n)
        for _ in range(n):
            ref.step(1)
        _same(many, ref, f"{block} threads, pipelined")
        _same(off, ref, f"{block} threads")


def test_pipelined_passes_on_the_large_workload():
    # 4M + 4M, ions sub-cycled x10: 23 steps in one call against single steps
    w = workloads.get("c3_large_lowp")
    many, ref = _passes(dict(w["params"], flags=RECORD), state.initial_state(w))
    _compare(many, ref, (23,), "large")


def test_capacity_overflow_in_pipelined_passes_is_reported():
    from paper_2109_04469_amd import Discharge, PicError

    w = workloads.scaled(workloads.get("c1_small"), 2000)
    p = dict(w["params"], capacity=(2000, 4000), pressure_pa=300.0, ion_subcycle=4, sort_interval=0)
    d = Discharge(p, xsec.argon_synthetic())
    d.timing(1)
    d.set_state(0, *state.maxwellian_uniform(2000, p["gap_m"], 50.0, 0, 3), step=0)
    d.set_state(1, *state.maxwellian_uniform(2000, p["gap_m"], 0.03, 1, 3), step=0)
    d.step(7)
    assert d.sync() == -3
    with pytest.raises(PicError):
        d.get_state(0)


@pytest.mark.parametrize("path", ["one kernel", "pipelined passes", "passes", "batch"])
@pytest.mark.parametrize("species,value", [(0, np.nan), (0, np.inf), (1, np.nan), (1, -np.inf)])
def test_states_that_are_not_finite_are_reported(path, species, value):
    import torch

    from paper_2109_04469_amd import Batch, Discharge

    w = workloads.scaled(workloads.get("c1_small"), 3000)
    p = dict(w["params"], ion_subcycle=2)
    init = state.initial_state(w, seed=4)
    d = Discharge(p, xsec.argon_synthetic(), stream=torch.cuda.current_stream())
    bad = [a.copy() for a in init[species]]
    bad[1][1234] = value
    for sp in (0, 1):
        d.set_state(sp, *(bad if sp == species else init[sp]), step=0)
    if path == "pipelined passes":
        d.timing(1)
    d.set_pipeline(path != "passes")
    b = Batch([d]) if path == "batch" else d
    b.step(3)
    assert d.sync() == -4
    for sp in (0, 1):
        d.set_state(sp, *init[sp], step=0)
    b.step(3)
    assert d.sync() == 0
