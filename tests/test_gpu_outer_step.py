"""The outer step's bookkeeping where the row chunks of the dot sweep go from its own sums to separate
reduction launches (16 and 17 chunks of 2048 rows, 8 and 9 at the segment edge), with one right-hand side
and several (the last workgroup advances the step), replayed from a graph and launched one by one, and over
restart cycles (a finished column without a following step).

Properties and bound as for the sweeps: an orthonormal basis, and a residual estimate equal to the
true residual, both to 1e-11.
"""

import numpy as np
import pytest

from tests.gpu_common import to_gpu
from tests.test_gpu_outer_shapes import test_outer_basis_and_residual as check_outer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.mark.parametrize("n,parts,nrhs,columns", [(181, 6, 1, 9), (183, 6, 1, 9), (128, 4, 2, 6), (130, 4, 3, 6)])
def test_chunk_edges(torch, n, parts, nrhs, columns):
    check_outer(torch, n, parts, nrhs, columns)


@pytest.mark.parametrize("nrhs", [1, 3])
def test_graph_and_restarts(torch, nrhs):
    """Replayed and eager steps give the same bits; restarted solves end with their true residual."""
    from paper_2103_17081_amd import inputs
    from paper_2103_17081_amd.binding import Solver
    n = 40
    f = np.stack([inputs.gaussian_load(n, inputs.gaussian_params(np.random.default_rng(q))) for q in range(nrhs)])
    f = to_gpu(torch, f if nrhs > 1 else f[0])
    for restart in (0, 5):
        us = []
        for graph in (1, 0):
            kw = dict(outer_restart=restart) if restart else {}
            with Solver(2 * np.pi * n / 20.0, n_intervals=n, px=2, py=2, local_solver="direct", nrhs=nrhs,
                        outer_maxit=17, outer_tol=1e-12, graph_steps=2, use_graph=graph, **kw) as s:
                for _ in range(3):
                    u, st = s.solve(f)
                us.append(u.clone())
                worst = max(float(torch.linalg.vector_norm(g - s.op_global_apply(v.contiguous())) /
                                  torch.linalg.vector_norm(g))
                            for g, v in zip(f.reshape(nrhs, -1), u.reshape(nrhs, -1)))
                assert abs(worst - st["final_res_estimate"]) <= 1e-11, (worst, st["final_res_estimate"])
        assert torch.equal(us[0], us[1])
