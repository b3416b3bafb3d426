"""The cell sort at the edges of its launches: particles around what a
workgroup scatters at a time, one chunk and more chunks than a wave scans at
once, the smallest and largest grids. Particles at rest in no field stay where
they are, so one step followed by a sort must give the stable order by cell
of the initial state, exactly; one discharge and a batch."""
import numpy as np
import pytest

from gpu_common import assert_state_equal, need_gpu
from helpers import NO_COLL, NO_FIELD
from pic_inputs import workloads, xsec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("n,cap,cells", [
    ((0, 1), 64, 2),
    ((2047, 2048), 4096, 64),
    ((2049, 4097), 4097, 255),
    ((5000, 4999), 5000, 4096),
    ((70001, 9), 300_000, 512),
])
def test_sort_is_the_stable_order_by_cell(n, cap, cells):
    import torch

    from paper_2109_04469_amd import Batch, Discharge

    p = dict(workloads.get("c1_small")["params"], n_cells=cells, capacity=(cap, cap),
             flags=NO_COLL | NO_FIELD, sort_interval=1, ion_subcycle=1)
    rng = np.random.default_rng(sum(n) + cells)
    s = torch.cuda.Stream()
    one, two, three = (Discharge(p, xsec.argon_synthetic(), stream=s) for _ in range(3))
    want = []
    for sp in (0, 1):
        x = rng.uniform(0.05, 0.95, n[sp]) * p["gap_m"]
        a = (x, np.zeros(n[sp]), rng.normal(size=n[sp]), rng.normal(size=n[sp]))
        for d in (one, two, three):
            d.set_state(sp, *a, step=0)
        cell = np.clip((x * (1.0 / (p["gap_m"] / cells))).astype(np.int64), 0, cells - 1)
        order = np.argsort(cell, kind="stable")
        want.append(tuple(v[order] for v in a))
    one.step(1)
    Batch([two, three]).step(1)
    for d in (one, two, three):
        assert d.sync() == 0
        for sp in (0, 1):
            assert_state_equal(d.get_state(sp), want[sp], f"species {sp}")


# particles of the largest of three unlike discharges sorted together: one
# chunk of each, two and four lanes per cell, more chunks than a wave scans at once
@pytest.mark.parametrize("n,cap,cells", [
    (2048, 2048, 64), (2049, 9000, 4096), (8193, 16384, 1200), (140_001, 300_000, 130),
])
def test_sorts_of_unlike_discharges_together(n, cap, cells):
    import torch

    from paper_2109_04469_amd import Batch, Discharge

    s = torch.cuda.Stream()
    ds, want = [], []
    for k, (ne, ni, c) in enumerate(((n, n // 3, cells), (1, 0, 2), (n // 2, n, cells // 2))):
        p = dict(workloads.get("c1_small")["params"], n_cells=c, capacity=(cap, cap),
                 flags=NO_COLL | NO_FIELD, sort_interval=1, ion_subcycle=1)
        rng = np.random.default_rng(n + k)
        d = Discharge(p, xsec.argon_synthetic(), stream=s)
        for sp, m in ((0, ne), (1, ni)):
            x = rng.uniform(0.05, 0.95, m) * p["gap_m"]
            a = (x, np.zeros(m), rng.normal(size=m), rng.normal(size=m))
            d.set_state(sp, *a, step=0)
            cell = np.clip((x * (1.0 / (p["gap_m"] / c))).astype(np.int64), 0, c - 1)
            order = np.argsort(cell, kind="stable")
            want.append(tuple(v[order] for v in a))
        ds.append(d)
    Batch(ds).step(1)
    for k, d in enumerate(ds):
        assert d.sync() == 0
        for sp in (0, 1):
            assert_state_equal(d.get_state(sp), want[2 * k + sp], f"discharge {k}, species {sp}")
