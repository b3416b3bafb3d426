"""The network's fused passes at their edges: each number of rows per
workgroup (batches up to 512, 1024, 2048 and beyond), rows, features and
layers that do not fill a 32 x 32 product, no hidden layer, the widest rows
the LDS takes and the first it does not (layer-by-layer kernels). Against the
CPU oracle: both round the same operands to BF16, so what differs is the FP32
accumulation and, rarely, an operand rounded the other way (2^-8 of one term
of a sum): 2e-3 of the largest output, 5e-3 of the largest gradient of a
tensor. A training step must equal the gradient followed by the optimiser,
and the call without a workspace the network's own forward pass, exactly."""
import numpy as np
import pytest

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu

SHAPES = [  # n_in, width, depth, n_out, batch
    (1, 1, 1, 1, 1),
    (33, 31, 3, 65, 31),
    (6, 64, 0, 45, 33),
    (5, 33, 1, 32, 513),
    (6, 40, 2, 7, 1025),
    (3, 32, 2, 33, 2049),
    (1024, 1024, 1, 1024, 3),
    (6, 1025, 1, 9, 5),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("shape", SHAPES)
def test_passes_match_oracle(shape):
    import torch

    from oracle import mlp
    from paper_2109_04469_amd import Mlp, mlp_forward_static

    n_in, width, depth, n_out, batch = shape
    rng = np.random.default_rng(sum(shape))
    dims = mlp.dims_of(n_in, width, depth, n_out)
    p = np.zeros(mlp.num_params(dims))
    for W, b in mlp.unpack(p, dims):
        W[...] = rng.normal(scale=np.sqrt(2.0 / W.shape[1]), size=W.shape)
        b[...] = rng.normal(scale=0.1, size=b.shape)
    p = p.astype(np.float32)
    x = rng.normal(size=(batch, n_in)).astype(np.float32)
    t = rng.normal(size=(batch, n_out)).astype(np.float32)
    xd, td = torch.as_tensor(x).cuda(), torch.as_tensor(t).cuda()

    one, two = Mlp(n_in, width, depth, n_out, batch), Mlp(n_in, width, depth, n_out, batch)
    one.set_params(p)
    two.set_params(p)
    y = one.forward(xd)
    yo, _ = mlp.forward(p, x, dims)
    assert np.abs(y.cpu().numpy() - yo).max() <= 2e-3 * np.abs(yo).max()
    ys = mlp_forward_static(shape[:4], torch.as_tensor(p).cuda(), xd)
    assert torch.equal(y, ys)

    loss, g = one.grad(xd, td)
    lo, go = mlp.loss_and_grad(p, x, t, dims)
    assert loss == pytest.approx(lo, rel=2e-3)
    for layer, ((gW, gb), (oW, ob)) in enumerate(zip(mlp.unpack(g, dims), mlp.unpack(go, dims))):
        for a, o in ((gW, oW), (gb, ob)):
            assert np.abs(a - o).max() <= 5e-3 * np.abs(o).max(), f"layer {layer}"

    for b in (batch, max(1, batch // 2)):
        one.grad(xd[:b], td[:b])
        one.adam(1e-3, weight_decay=0.01)
        two.train_step(xd[:b], td[:b], 1e-3, weight_decay=0.01)
        assert one.loss() == two.loss()
    assert np.array_equal(one.get_params(), two.get_params())
    assert torch.equal(one.forward(xd), two.forward(xd))


def test_results_over_the_inputs():
    # y may lie over x: two rows of results share memory with later inputs
    import ctypes

    import torch

    from paper_2109_04469_amd import Mlp, capi

    net = Mlp(4, 32, 1, 6, 1100)
    net.set_params(np.random.default_rng(2).normal(size=net.num_params).astype(np.float32))
    x = torch.randn(1100, 4, device="cuda")
    want = net.forward(x)
    mem = torch.zeros(1100 * 6, device="cuda")
    mem[:1100 * 4] = x.reshape(-1)
    torch.cuda.synchronize()
    p = ctypes.c_void_p(mem.data_ptr())
    assert net.L.pic_mlp_forward(net.h, p, 1100, p) == capi.PIC_OK
    torch.cuda.synchronize()
    assert torch.equal(mem.reshape(1100, 6), want)
