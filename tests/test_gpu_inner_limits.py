"""Subdomain GMRES on the smallest tiles with the longest bases that fit in LDS, against the oracle.

Tiles of 2 x 2 to 3 x 3 nodes are smaller than the coarse solve's scratch: the scratch then lies in another
vector of the solve (62 iterations and more) or takes extra room (61).  652 and 968 are the largest iteration limits
that such tiles have room for without the scratch.

Bounds: those of the other subdomain-solve tests (1e-8 for complex128 at equal counts; 2e-3 for complex64 at
tolerance 1e-4)."""

import numpy as np
import pytest

from oracle import schwarz
from tests.gpu_common import crandn, pack, to_gpu, to_np, unpack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.mark.parametrize("prec,maxit", [(64, 652), (64, 62), (64, 61), (32, 968), (32, 61)])
def test_smallest_tiles_longest_bases(torch, prec, maxit):
    from paper_2103_17081_amd.binding import Solver
    print("case: smallest tiles", prec, maxit, flush=True)
    k, n, cuts = 5.0, 8, [0, 2, 4, 6, 8]
    S = schwarz.Schwarz(schwarz.Problem(k, n, np.asarray(cuts), np.asarray(cuts), local_bc="dirichlet"))
    tol = 1e-10 if prec == 64 else 1e-4
    with Solver(k, n_intervals=n, cuts_x=cuts, cuts_y=cuts, local_bc="dirichlet", inner_precision=prec, inner_tol=tol,
                inner_maxit=maxit, outer_maxit=2) as gpu:
        assert (gpu.layout[:, 2].max(), gpu.layout[:, 3].max()) == (3, 3)
        rng = np.random.default_rng(7)
        fs = [crandn(rng, s.geom.ndof) for s in S.subs]
        packed = pack(S, gpu, fs).astype(np.complex64 if prec == 32 else np.complex128)
        u, iters, _ = gpu.op_inner_solve(to_gpu(torch, packed))
        us = unpack(S, gpu, to_np(u).astype(np.complex128))
    for s, f, ug, it in zip(S.subs, fs, us, iters):
        ur, itr, _ = s.deflated_gmres(f, tol, maxit)
        assert abs(int(it) - itr) <= 1
        if it == itr:
            assert np.linalg.norm(ug - ur) <= (1e-8 if prec == 64 else 2e-3) * np.linalg.norm(ur)
