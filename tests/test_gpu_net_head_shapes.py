"""Loss and gradient where the strips of rows of the head's training kernels can go wrong, against the
float64 oracle: subdomains of one and two rows, up to the last row of a strip, one row into the next, and the
whole tile; tiles of 32 to 128 and 16 to 32 head channels; sides that are subdomain edges or not (two
opposite edges are at least two rows apart: the operator has no cells otherwise); an empty target (zero
denominators).

Bounds of the other gradient tests, 2e-2 for the loss and 5e-2 per parameter tensor, for the head's
parameters and those of the layer that its gradient reaches first.  (Deeper layers see a few noisy
pixels of a small subdomain through every bfloat16 rounding of the backward pass; their kernels are
tested on whole tiles.)
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


def _operator(nx, ny, edges, robin, kh):
    """The subdomain operator on its nodes: a rectangle with a ring of cells on the sides that are no edges."""
    from perf.cases import _rectangle
    w, s = (0 if edges & 1 else 1), (0 if edges & 4 else 1)
    fx, fy = nx + w + (0 if edges & 2 else 1), ny + s + (0 if edges & 8 else 1)
    keep = np.arange(fx * fy).reshape(fy, fx)[s:s + ny, w:w + nx].ravel()
    return _rectangle(fx, fy, kh, robin)[np.ix_(keep, keep)]


def _gradient(torch, widths, x, t, sizes, edges, w_res, w_err, v):
    from paper_2103_17081_amd.binding import GuessNet, TileDesc
    ds = (TileDesc * len(sizes))()
    for d, (nx, ny) in zip(ds, sizes):
        d.nx, d.ny, d.edges, d.robin, d.kh = nx, ny, edges, edges, 0.4
    net = GuessNet(widths, tile=x.shape[1], max_batch=len(sizes), train=True)
    net.set_params(v.astype(np.float32))
    loss, g = net.gradient(to_gpu(torch, x.astype(np.float32)), to_gpu(torch, t.astype(np.float32)), ds,
                           w_res=w_res, w_err=w_err, want_grad=True)
    g = to_np(g).astype(np.float64)
    net.close()
    return loss, g


@pytest.mark.parametrize("widths,tile,sizes,edges", [
    ((16, 16, 16, 16), 32, [(5, 2), (32, 8), (7, 9), (32, 32)], 15),
    ((16, 32, 64, 64), 64, [(40, 16), (17, 33), (11, 1)], 6),
    ((32, 32, 32, 32), 64, [(33, 24)], 0),
    ((16, 16, 32, 32), 128, [(30, 31), (9, 128)], 15),
])
def test_loss_and_gradient(torch, widths, tile, sizes, edges):
    print("case:", widths, tile, sizes, edges, flush=True)
    rng = np.random.default_rng(tile + edges)
    x = bf16_round(rng.standard_normal((len(sizes), tile, tile, 4)))
    t = rng.standard_normal((len(sizes), tile, tile, 2)).astype(np.float32).astype(np.float64)
    v = oracle_params(11, widths)
    loss, g = _gradient(torch, widths, x, t, sizes, edges, 0.3, 1.0, v)
    p = cnn.unflatten(v, widths)
    y, c = cnn.forward(p, x)
    lo, dy = 0.0, np.zeros_like(y)
    for b, (nx, ny) in enumerate(sizes):
        B = _operator(nx, ny, edges, edges, 0.4)
        e = (y - t)[b, :ny, :nx, 0].ravel() + 1j * (y - t)[b, :ny, :nx, 1].ravel()
        tt = t[b, :ny, :nx, 0].ravel() + 1j * t[b, :ny, :nx, 1].ravel()
        r, res, err = B @ e, np.vdot(B @ tt, B @ tt).real, np.vdot(tt, tt).real
        lo += (0.3 * np.vdot(r, r).real / res + np.vdot(e, e).real / err) / len(sizes)
        q = (2 * 0.3 * (B.conj().T @ r) / res + 2 * e / err) / len(sizes)
        dy[b, :ny, :nx, 0], dy[b, :ny, :nx, 1] = q.real.reshape(ny, nx), q.imag.reshape(ny, nx)
    go = cnn.flatten(cnn.backward(p, c, dy))
    assert abs(loss - lo) <= 2e-2 * lo
    gp, gop = cnn.unflatten(g, widths), cnn.unflatten(go, widths)
    for k in ("W8", "b8", "W7", "b7"):
        assert rel(gp[k], gop[k]) <= 5e-2, (k, rel(gp[k], gop[k]))


def test_empty_target(torch):
    """Zero denominators count as one: the loss is the mean of ||y||^2 over the nodes of each tile."""
    widths, tile = (16, 16, 16, 16), 32
    x = bf16_round(np.random.default_rng(1).standard_normal((2, tile, tile, 4)))
    v = oracle_params(11, widths)
    loss, g = _gradient(torch, widths, x, np.zeros((2, tile, tile, 2)), [(20, 20), (9, 30)], 15, 0.0, 1.0, v)
    y, _ = cnn.forward(cnn.unflatten(v, widths), x)
    lo = 0.5 * (np.sum(y[0, :20, :20] ** 2) + np.sum(y[1, :30, :9] ** 2))
    assert abs(loss - lo) <= 2e-2 * lo and np.all(np.isfinite(g))
