"""The network's forward pass on rows that hold infinities or overflow, at
layer widths that do and do not fill a 32-feature tile. With positive weights
every product of such a row is +inf, so its outputs are +inf, exactly as plain
FP32 arithmetic gives them, and the rows beside it are those of a batch
without it, exactly: a row's products are its own."""
import numpy as np
import pytest

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("dims", [(6, 33, 2, 45), (5, 31, 3, 32), (33, 64, 1, 7), (6, 1025, 1, 9)])
@pytest.mark.parametrize("value", [np.inf, 3.0e38])
def test_infinite_rows_stay_infinite_and_apart(dims, value):
    import torch

    from paper_2109_04469_amd import Mlp, mlp_forward_static

    n_in, width, depth, n_out = dims
    batch, bad = 37, 5
    rng = np.random.default_rng(sum(dims))
    net = Mlp(*dims, batch)
    p = rng.uniform(1.0, 2.0, net.num_params).astype(np.float32)
    net.set_params(p)
    x = rng.uniform(0.0, 1.0, (batch, n_in)).astype(np.float32)
    want = net.forward(x).cpu().numpy()
    x[bad, 0] = value
    want[bad] = np.inf
    assert np.array_equal(net.forward(x).cpu().numpy(), want)
    ys = mlp_forward_static(dims, torch.as_tensor(p).cuda(), torch.as_tensor(x).cuda())
    assert np.array_equal(ys.cpu().numpy(), want)
