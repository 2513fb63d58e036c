"""Exact local solves at the tile widths where their form changes: 16 and 17, 26 and 27, 32 and 33, 40 and 41, 48 and 49 nodes,
narrow tiles, and a tall tile whose couplings do not fit the wave chain's LDS.

Bound: an FP64 elimination of a well-posed local matrix, ||B u - f|| <= 1e-10 ||f|| as in the other
tests of the exact solves.
"""

import numpy as np
import pytest

from tests.gpu_common import crandn, to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.mark.parametrize("wide", [4, 5, 16, 17, 26, 27, 32, 33, 40, 41, 48, 49])
@pytest.mark.parametrize("bc", ["impedance", "dirichlet"])
def test_direct_forms(torch, wide, bc):
    from paper_2103_17081_amd.binding import Solver
    print("case:", wide, bc, flush=True)
    grow = 3 if bc == "impedance" else 1
    w = wide - grow                                   # cells of the middle block
    cx = cy = [0, 2, 2 + w, 4 + w]
    with Solver(0.35 * (4 + w), n_intervals=4 + w, cuts_x=cx, cuts_y=cy, local_bc=bc, local_solver="direct",
                outer_maxit=2) as s:
        f = to_gpu(torch, crandn(np.random.default_rng(wide), s.nfine))
        u, _, _ = s.op_inner_solve(f)
        r = s.op_local_apply(u) - f
        assert float(torch.linalg.vector_norm(r) / torch.linalg.vector_norm(f)) <= 1e-10


def test_direct_tall_tiles(torch):
    from paper_2103_17081_amd.binding import Solver
    n = 128                                           # strips of 16 cells: 19 x 127 nodes
    with Solver(0.3 * n, n_intervals=n, cuts_x=list(range(0, n + 1, 16)), cuts_y=[0, n], local_solver="direct",
                outer_maxit=2) as s:
        f = to_gpu(torch, crandn(np.random.default_rng(1), s.nfine))
        u, _, _ = s.op_inner_solve(f)
        r = s.op_local_apply(u) - f
        assert float(torch.linalg.vector_norm(r) / torch.linalg.vector_norm(f)) <= 1e-10
