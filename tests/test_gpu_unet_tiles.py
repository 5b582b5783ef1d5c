"""The network's gradient kernels at the edges of their tiles: levels whose
x rows are shorter than a 16-voxel tile or end inside one, whose y and z
extents are odd or below a tile, and grids of many tiles per workgroup."""
import numpy as np
import pytest

from . import unet_bf16 as B
from .test_gpu_unet import grad_checks, model_samples, params, rel
from oracle import unet as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 24, 40), (16, 40, 24), (24, 8, 48)])
def test_gradients_on_ragged_levels(gpu_lib, shape):
    """Against the FP64 oracle within reach of the BF16 model (the bounds of
    the gradient test at 16x16x32)."""
    from paper_2606_05893_amd.pic import UNet
    p = params(5)
    rng = np.random.default_rng(sum(shape))
    x = rng.standard_normal(shape + (2,)).astype(np.float32)
    t = rng.standard_normal(shape).astype(np.float32)
    g, loss = UNet(*shape, params=p).gradients(x, t)
    loss_o, g_o, _ = U.loss_and_grad(p.astype(np.float64), x.astype(np.float64), t.astype(np.float64))
    g_ms = model_samples(p, lambda q: B.loss_and_grad(q, x, t)[1])
    assert abs(loss - loss_o) <= 0.02 * loss_o
    print(shape, grad_checks(g.cpu().numpy().astype(np.float64), g_o, g_ms, str(shape)))


def test_gradients_equivariant_under_rolls(gpu_lib):
    """x and y are periodic and every activation and gradient value is the
    rolled one bit for bit when the sample is rolled by multiples of 8 voxels,
    so each parameter's gradient is the same sum in another order.  FP32 sums
    of V = 1e5 products of either sign, about sqrt(V) times smaller than their
    absolute sum: 6e-8 sqrt(V) = 2e-5 relative in a random order, bound 2e-4."""
    from paper_2606_05893_amd.pic import UNet
    shape = (16, 72, 88)
    p = params(6)
    net = UNet(*shape, params=p)
    rng = np.random.default_rng(2)
    x = rng.standard_normal(shape + (2,)).astype(np.float32)
    t = rng.standard_normal(shape).astype(np.float32)
    g = net.gradients(x, t)[0].cpu().numpy().astype(np.float64)
    for sy, sx in ((8, 0), (0, 24), (32, 40)):
        gr = net.gradients(np.roll(x, (sy, sx), (1, 2)), np.roll(t, (sy, sx), (1, 2)))[0]
        gr = gr.cpu().numpy().astype(np.float64)
        for name, kind, off, shp in U.param_layout()[0]:
            sl = slice(off, off + int(np.prod(shp)))
            assert rel(gr[sl], g[sl]) <= 2e-4, (sy, sx, name, kind, rel(gr[sl], g[sl]))
