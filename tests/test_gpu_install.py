"""A species replaced (pic_set_state from host and from device arrays,
pic_load_profile) at the edges of its launches: sizes around one workgroup's
share, the smallest and largest grids, profiles whose table fills the LDS
beside the deposit's and ones that leave it no room, and a step index of the
other parity. Positions, velocities and the 2^-32 fixed-point deposit are
compared exactly with the CPU's (same FP64 operations, integer sums), loaded
velocities at the 1e-12 of their logarithms and cosines."""
import numpy as np
import pytest

from gpu_common import assert_state_equal, need_gpu
from helpers import MAR, ME, QE
from pic_inputs import workloads, xsec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _params(cells, n):
    w = workloads.scaled(workloads.get("c1_small"), max(n, 16), capacity_factor=3)
    return dict(w["params"], n_cells=cells)


def _deposit(x, gap, cells):
    """2^-32 fixed-point linear weights, the largest rounding to nearest."""
    t = x * (1.0 / (gap / cells))
    j = np.clip(t.astype(np.int64), 0, cells - 1)
    w = np.clip(np.floor((t - j) * 2.0**32 + 0.5), 0.0, 2.0**32).astype(np.int64)
    d = np.zeros(cells + 1, np.int64)
    np.add.at(d, j, 2**32 - w)
    np.add.at(d, j + 1, w)
    return d


@pytest.mark.parametrize("device_arrays", [False, True])
@pytest.mark.parametrize("n,cells", [(0, 2), (1, 2), (1023, 64), (1025, 4096), (70001, 255)])
def test_set_state_arrays_and_deposit(n, cells, device_arrays):
    import torch

    from paper_2109_04469_amd import Discharge

    p = _params(cells, n)
    rng = np.random.default_rng(n + cells)
    d = Discharge(p, xsec.argon_synthetic())
    for step, sp in ((0, 0), (3, 1), (4, 0)):
        a = (rng.uniform(0, p["gap_m"], n), *rng.normal(size=(3, n)))
        if n > 1:
            a[0][:2] = 0.0, p["gap_m"]
        src = [torch.as_tensor(v).cuda() for v in a] if device_arrays else a
        d.set_state(sp, *src, step=step)
        assert_state_equal(d.get_state(sp), a, f"species {sp}")
        assert d.step_index == step
        assert np.array_equal(d.get_field()["dep_e" if sp == 0 else "dep_i"],
                              _deposit(a[0], p["gap_m"], cells))


@pytest.mark.parametrize("n,cells,npts", [(1, 2, 2), (1025, 64, 9), (5000, 4096, 4095),
                                          (5000, 4096, 4096), (3001, 100, 8192)])
def test_load_profile_state_and_deposit(n, cells, npts):
    import oracle

    from paper_2109_04469_amd import Discharge

    p = _params(cells, n)
    rng = np.random.default_rng(npts)
    d = Discharge(p, xsec.argon_synthetic())
    dens, temp = rng.uniform(0, 2, npts), rng.uniform(1, 4, npts)
    for sp, m in ((0, ME), (1, MAR)):
        d.load_profile(sp, n, dens, temp, step=sp)
        g = d.get_state(sp)
        o = oracle.load_profile(dens, temp, p["gap_m"], QE / m, p["seed"], p["run"], sp, n)
        assert np.array_equal(g[0], o[0])
        for k in (1, 2, 3):
            np.testing.assert_allclose(g[k], o[k], rtol=1e-12, atol=1e-12 * np.abs(o[k]).max())
        assert np.array_equal(d.get_field()["dep_e" if sp == 0 else "dep_i"],
                              _deposit(g[0], p["gap_m"], cells))
