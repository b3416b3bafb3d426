"""What the reading calls may be given to write to: the caller's host memory,
its own GPU's arrays, arrays that are not 8-byte aligned and memory that both
sides reach. All hold the same bytes as host arrays get."""
import ctypes

import numpy as np
import pytest

from gpu_common import need_gpu
from pic_inputs import state, workloads, xsec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _discharge(stream=None):
    from paper_2109_04469_amd import Discharge

    w = workloads.scaled(workloads.get("c1_small"), 2000)
    d = Discharge(w["params"], xsec.argon_synthetic(), stream=stream)
    init = state.initial_state(w, seed=3)
    for sp in (0, 1):
        d.set_state(sp, *init[sp], step=0)
    d.step(5)
    return d


@pytest.mark.parametrize("where", ["device", "misaligned device", "pinned", "mixed"])
def test_field_arrays_may_lie_anywhere(where):
    import torch

    d = _discharge()
    want = d.get_field()
    nbytes = 8 * d.nx
    ptrs, bufs = [], []
    for k in range(5):
        if where == "pinned":
            b = torch.zeros(nbytes, dtype=torch.uint8, pin_memory=True)
        elif where == "mixed" and k % 2:
            b = torch.zeros(nbytes, dtype=torch.uint8)
        else:
            b = torch.zeros(nbytes + 4, dtype=torch.uint8, device="cuda")
            b = b[4:] if where == "misaligned device" or k == 2 else b[:nbytes]
        bufs.append(b)
        ptrs.append(ctypes.c_void_p(b.data_ptr()))
    torch.cuda.synchronize()
    assert d.L.pic_get_field(d.h, *ptrs) == 0
    for k, name in enumerate(("rho", "phi", "E", "dep_e", "dep_i")):
        got = bufs[k].cpu().numpy().tobytes()
        assert got == np.ascontiguousarray(want[name]).tobytes(), name
