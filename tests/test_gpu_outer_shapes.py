"""Outer orthogonalisation at the grid sizes where the shape of its update sweep changes: fewer
2048-row chunks than compute units (sliced basis, one row per lane), one chunk per compute unit
(chunk kernel), more chunks than compute units (sliced, four rows per lane); basis lengths
below, at and above the 8 slices; remainders of rows in every case.

Two properties of the flexible Arnoldi process pin every output of the sweep: the finished basis is
orthonormal, and the residual estimate of the rotated Hessenberg matrix is the true residual of
the returned iterate.  Both hold to FP64 rounding (a few units per column and 1e6 entries:
1e-11 leaves two orders).
"""

import numpy as np
import pytest

from tests.gpu_common import to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.mark.parametrize("n,parts,nrhs,columns", [(33, 2, 1, 20), (33, 2, 3, 7), (160, 8, 1, 9), (594, 16, 1, 17),
                                                  (760, 20, 1, 17), (420, 12, 4, 8)])
def test_outer_basis_and_residual(torch, n, parts, nrhs, columns):
    print("case: outer shapes", n, parts, nrhs, columns, flush=True)
    from paper_2103_17081_amd import inputs
    from paper_2103_17081_amd.binding import Solver
    fs = []
    for q in range(nrhs):
        rng = np.random.default_rng(100 + q)
        fs.append(inputs.gaussian_load(n, inputs.gaussian_params(rng)))
    f = to_gpu(torch, np.stack(fs) if nrhs > 1 else fs[0])
    with Solver(2 * np.pi * n / 20.0, n_intervals=n, px=parts, py=parts, local_solver="direct", nrhs=nrhs,
                outer_maxit=columns, outer_tol=1e-12, graph_steps=4) as s:
        u, st = s.solve(f)
        assert st["status"] == "DD_ENOTCONV" and st["outer_iters"] == columns
        V = torch.stack([s.outer_basis(j).reshape(nrhs, -1) for j in range(columns)])
        worst = 0.0
        for q in range(nrhs):
            w = s.op_global_apply(u.reshape(nrhs, -1)[q].contiguous())
            fq = f.reshape(nrhs, -1)[q]
            worst = max(worst, float(torch.linalg.vector_norm(fq - w) / torch.linalg.vector_norm(fq)))
            Vq = V[:, q].contiguous()
            gram = torch.stack([torch.stack([torch.vdot(a, b) for b in Vq]) for a in Vq])
            err = float((gram - torch.eye(columns, dtype=gram.dtype, device=gram.device)).abs().max())
            assert err <= 1e-11, (q, err)
        assert abs(worst - st["final_res_estimate"]) <= 1e-11, (worst, st["final_res_estimate"])
