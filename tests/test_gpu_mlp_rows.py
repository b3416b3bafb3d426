"""Predictions of more rows than 32 per compute unit, where a workgroup's waves
follow the layers' widths: narrow and mixed layers, wide inputs, no hidden
layer, a last workgroup that is not full. A row's products are its own and are
summed in one order however the rows are dealt, so the results equal those of
500 rows at a time exactly."""
import numpy as np
import pytest

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("dims", [(6, 32, 2, 32), (6, 16, 1, 1), (6, 33, 3, 512), (300, 40, 1, 7),
                                  (1024, 64, 0, 5), (6, 200, 2, 65)])
@pytest.mark.parametrize("batch", [8193, 40_001])
def test_many_rows_equal_few_rows(dims, batch):
    import torch

    from paper_2109_04469_amd import Mlp

    rng = np.random.default_rng(batch + sum(dims))
    many, few = Mlp(*dims, batch), Mlp(*dims, 500)
    p = rng.normal(scale=0.1, size=many.num_params).astype(np.float32)
    many.set_params(p)
    few.set_params(p)
    x = torch.as_tensor(rng.normal(size=(batch, dims[0])).astype(np.float32)).cuda()
    y = many.forward(x)
    for i in range(0, batch, 500):
        assert torch.equal(y[i:i + 500], few.forward(x[i:i + 500])), i
