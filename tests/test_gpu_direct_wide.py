"""Exact local solves where the step-by-step forms change: 55 to 57, 61, 64 and 65 nodes (columns per lane, the plain
form), a handle that mixes them with narrow tiles, tall narrow tiles (couplings formed as the chain goes: 5, 18, 31 nodes
wide), and a tile that leaves no LDS for a vector per wave.  Subdomain GMRES with coarse blocks of 27 to 32 unknowns per row.

Bounds: an FP64 elimination of a well-posed local matrix, ||B u - f|| <= 1e-10 ||f||, and the coarse solve's 1e-9
against the oracle, as in the other tests of these solves."""

import numpy as np
import pytest

from oracle import schwarz
from tests.gpu_common import crandn, pack_coarse, to_gpu, to_np, unpack_coarse

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.mark.parametrize("cx,cy,widest", [
    ([0, 54, 60], [0, 20, 60], 55), ([0, 55, 62], [0, 20, 62], 56), ([0, 56, 62], [0, 20, 62], 57),
    ([0, 60, 66], [0, 20, 66], 61), ([0, 63, 72], [0, 20, 72], 64), ([0, 64, 72], [0, 20, 72], 65),
    ([0, 2, 10, 40, 80], [0, 2, 10, 40, 80], 41),
    (list(range(0, 421, 2)), [0, 420], 5), (list(range(0, 129, 15)) + [128], [0, 128], 18), (list(range(0, 141, 28)), [0, 140], 31),
    ([0, 61, 80], [0, 80], 62)])
def test_wide_and_tall_tiles(torch, cx, cy, widest):
    from paper_2103_17081_amd.binding import Solver
    print("case: direct", widest, cx, cy, flush=True)
    n = cx[-1]
    for bc in ("impedance", "dirichlet"):
        with Solver(0.3 * n, n_intervals=n, cuts_x=cx, cuts_y=cy, local_bc=bc, local_solver="direct", outer_maxit=2) as s:
            if bc == "impedance":
                assert int(s.layout[:, 2].max()) == widest
            f = to_gpu(torch, crandn(np.random.default_rng(widest), s.nfine))
            u, _, _ = s.op_inner_solve(f)
            r = s.op_local_apply(u) - f
            assert float(torch.linalg.vector_norm(r) / torch.linalg.vector_norm(f)) <= 1e-10


@pytest.mark.parametrize("w", [53, 58, 63])
def test_coarse_blocks_past_the_chain(torch, w):
    from paper_2103_17081_amd.binding import Solver
    print("case: coarse blocks", (w + 1) // 2, flush=True)
    k, n, cx, cy = 30.0, w + 7, [0, w, w + 7], [0, 20, w + 7]
    S = schwarz.Schwarz(schwarz.Problem(k, n, np.asarray(cx), np.asarray(cy)))
    with Solver(k, n_intervals=n, cuts_x=cx, cuts_y=cy, inner_precision=32, inner_maxit=10, outer_maxit=2) as gpu:
        assert int(gpu.layout[:, 8].max()) == (w + 1) // 2
        rng = np.random.default_rng(w)
        ys = [crandn(rng, s.defl.ncoarse) for s in S.subs]
        sol = unpack_coarse(S, gpu, to_np(gpu.op_coarse_solve(to_gpu(torch, pack_coarse(S, gpu, ys)))))
    for s, y, x in zip(S.subs, ys, sol):
        ref = s.defl.coarse_solve(y)
        assert np.linalg.norm(x - ref) <= 1e-9 * np.linalg.norm(ref)
