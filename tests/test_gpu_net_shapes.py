"""Weight gradients at the shapes where their kernels change, against the float64 oracle.

Input channel blocks of 8 (the network input, half a block), 16, 32 (waves split the pixels), 64 and
128 (two windows); 16, 32 and 64 output channels; tiles of 32 (a last level of 16 pixels, half a product
step) to 128 (bands of a few rows); batches of one tile, of an odd number, and of more bands than
workgroups keep partials (513 tiles of a 128-channel layer: several bands each).

Bound: the network's activations and activation gradients are bfloat16, 5e-2 per parameter tensor and
a cosine of 0.999, as in the other gradient tests.  The loss is a mean over the tiles, so a batch of
equal tiles has the gradient of one of them.
"""

import numpy as np
import pytest

from oracle import cnn
from tests.gpu_common import to_gpu, to_np
from tests.test_gpu_net import bf16_round, oracle_params, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def _batch(tile, batch, rng):
    x = bf16_round(rng.standard_normal((batch, tile, tile, 4)))
    return x, rng.standard_normal((batch, tile, tile, 2)).astype(np.float32).astype(np.float64)


def _descs(tile, batch):
    from paper_2103_17081_amd.binding import TileDesc
    ds = (TileDesc * batch)()
    for d in ds:
        d.nx, d.ny, d.edges, d.robin, d.kh = tile, tile, 0, 0, 0.5
    return ds


def _gradient(torch, widths, v, x, t):
    from paper_2103_17081_amd.binding import GuessNet
    net = GuessNet(widths, tile=x.shape[1], max_batch=x.shape[0], train=True)
    net.set_params(v.astype(np.float32))
    _, g = net.gradient(to_gpu(torch, x.astype(np.float32)), to_gpu(torch, t.astype(np.float32)),
                        _descs(x.shape[1], x.shape[0]), w_res=0.0, w_err=1.0, want_grad=True)
    net.close()
    return to_np(g).astype(np.float64)


def _check(g, v, widths, x, t):
    p = cnn.unflatten(v, widths)
    y, c = cnn.forward(p, x)
    # the error term alone: mean over tiles of |y - t|^2 / |t|^2
    dy = 2.0 * (y - t) / np.sum(t * t, axis=(1, 2, 3), keepdims=True) / x.shape[0]
    go = cnn.flatten(cnn.backward(p, c, dy))
    gp, gop = cnn.unflatten(g, widths), cnn.unflatten(go, widths)
    for k in gop:
        assert rel(gp[k], gop[k]) <= 5e-2, (k, rel(gp[k], gop[k]))
    assert np.dot(g, go) / (np.linalg.norm(g) * np.linalg.norm(go)) >= 0.999


@pytest.mark.parametrize("widths,tile,batch", [
    ((16, 16, 16, 16), 32, 1), ((16, 32, 64, 64), 32, 3), ((16, 32, 64, 64), 64, 1), ((32, 64, 32, 32), 32, 2),
    ((16, 16, 32, 32), 128, 1),
])
def test_weight_gradients(torch, widths, tile, batch):
    print("case:", widths, tile, batch, flush=True)
    x, t = _batch(tile, batch, np.random.default_rng(tile + batch))
    v = oracle_params(11, widths)
    _check(_gradient(torch, widths, v, x, t), v, widths, x, t)


@pytest.mark.parametrize("batch", [33, 513])
def test_weight_gradients_of_equal_tiles(torch, batch):
    print("case:", batch, flush=True)
    widths = (16, 32, 64, 64)
    x, t = _batch(32, 1, np.random.default_rng(2))
    v = oracle_params(11, widths)
    _check(_gradient(torch, widths, v, np.repeat(x, batch, 0), np.repeat(t, batch, 0)), v, widths, x, t)
