"""Forward pass at the shapes where its kernels change, against the float64 oracle.

A last level of 16 pixels (one fragment of a workgroup's four), tiles of 128 (a workgroup takes half a
row), channel counts below and above one product step (16 and 32), and batches on both sides of the
choice of fragments per wave.

Bounds: 3e-2 per tile, as in the other network tests (7 layers rounded to bfloat16).  A tile's
products and sums are taken in the same order whatever the batch, so its output has the same bits.
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


@pytest.mark.parametrize("widths,tile,batch", [
    ((16, 16, 16, 16), 32, 40), ((16, 32, 64, 64), 32, 513), ((32, 64, 32, 32), 64, 35), ((16, 32, 64, 64), 64, 130),
    ((32, 32, 32, 32), 128, 9), ((16, 16, 32, 32), 128, 33),
])
def test_forward_shapes(torch, widths, tile, batch):
    from paper_2103_17081_amd.binding import GuessNet
    print("case:", widths, tile, batch, flush=True)
    x = bf16_round(np.random.default_rng(tile + batch).standard_normal((1, tile, tile, 4)))
    v = oracle_params(7, widths)
    net = GuessNet(widths, tile=tile, max_batch=batch)
    net.set_params(v.astype(np.float32))
    one = to_np(net.forward(to_gpu(torch, x.astype(np.float32))))
    many = to_np(net.forward(to_gpu(torch, np.repeat(x, batch, 0).astype(np.float32))))
    net.close()
    assert rel(one[0], cnn.forward(cnn.unflatten(v, widths), x)[0][0]) <= 3e-2
    assert np.array_equal(many, np.repeat(one, batch, 0))


def test_largest_layer_is_refused(torch):
    from paper_2103_17081_amd.binding import DDError, GuessNet
    net = GuessNet((64, 64, 64, 64), tile=32, max_batch=1)     # 128 channels into 64
    with pytest.raises(DDError):
        net.forward(torch.zeros((1, 32, 32, 4), device="cuda"))
    net.close()
