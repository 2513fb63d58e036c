"""Subdomain GMRES at the limits of its bases: the smallest tiles with the longest bases that fit in LDS, against
the oracle, and the byte count of bases longer than an update sweep holds.

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


@pytest.mark.parametrize("prec,maxit", [(64, 8), (64, 9), (64, 10), (64, 40), (32, 17), (32, 18), (32, 40)])
def test_bytes_of_long_bases(torch, prec, maxit):
    """The byte count of one subdomain solve (one subdomain, one outer step) that runs to its iteration limit, below and above
    the number of vectors (8, complex64 16) that the update sweep keeps for the next step's products."""
    from paper_2103_17081_amd.binding import Solver
    print("case: bytes of long bases", prec, maxit, flush=True)
    with Solver(30.0, n_intervals=24, cuts_x=[0, 24], cuts_y=[0, 24], inner_precision=prec, inner_tol=1e-12,
                inner_maxit=maxit, outer_maxit=1) as gpu:
        nx, ny, mx, my = (int(gpu.layout[0, c]) for c in (2, 3, 8, 9))
        f = crandn(np.random.default_rng(3), nx * ny)
        _, st = gpu.solve(to_gpu(torch, f))
    n, nc, k, s = nx * ny, mx * my, maxit, 8 if prec == 32 else 16
    assert st["precond_applies"] == 1 and st["inner_iters_total"] == k
    held = 16 if prec == 32 else 8
    basis_reads = sum((j + 1) + (j + 1) + max(0, j - held) for j in range(k))
    want = (16 * n + 16 * n + 16 * (k + 1) * (my * mx * mx + 3 * mx * my) + 16 * nc * (2 * k + 2) +
            s * n * (1 + 3 * k + basis_reads) + 2 * s * n)
    assert st["inner_bytes"] == want


@pytest.mark.parametrize("prec,k,n,tol,least", [(64, 80.0, 48, 1e-4, 80), (64, 80.0, 48, 1e-8, 115), (64, 100.0, 60, 1e-8, 150),
                                                (32, 80.0, 48, 1e-4, 80), (32, 100.0, 60, 1e-4, 100)])
def test_more_iterations_than_lanes(torch, prec, k, n, tol, least):
    """Solves of 80 to 163 iterations on under-resolved tiles of 25 and 31 nodes: the bookkeeping by one wave goes
    in two and three batches of 64.  Complex128 at equal counts agrees to 1e-8; in complex64 the residual that the solve
    stopped at is 2 tol at most in 64 bits (100 steps of 6e-8 on top of tol)."""
    from paper_2103_17081_amd.binding import Solver
    print("case: long solves", prec, k, tol, flush=True)
    cuts = [0, n // 2, n]
    S = schwarz.Schwarz(schwarz.Problem(k, n, np.asarray(cuts), np.asarray(cuts)))
    with Solver(k, n_intervals=n, cuts_x=cuts, cuts_y=cuts, inner_precision=prec, inner_tol=tol, inner_maxit=200,
                outer_maxit=2) as gpu:
        rng = np.random.default_rng(42)
        fs = [crandn(rng, s.geom.ndof) for s in S.subs]
        packed = pack(S, gpu, fs).astype(np.complex64 if prec == 32 else np.complex128)
        u, iters, flags = gpu.op_inner_solve(to_gpu(torch, packed))
        us = unpack(S, gpu, to_np(u).astype(np.complex128))
    for s, f, ug, it in zip(S.subs, fs, us, iters):
        d = s.defl
        ur, itr, _ = s.deflated_gmres(f, tol, 200)
        print("iterations", int(it), itr, flush=True)
        assert itr >= least and abs(int(it) - itr) <= 1
        if prec == 32:
            assert np.linalg.norm(d.P(f - s.B @ ug)) <= 2 * tol * np.linalg.norm(d.P(f))
        elif it == itr:
            assert np.linalg.norm(ug - ur) <= 1e-8 * np.linalg.norm(ur)


@pytest.mark.parametrize("prec,cells,maxit", [(64, 52, 100), (32, 66, 30)])
def test_largest_tiles(torch, prec, cells, maxit):
    """Tiles that fit in LDS because the coarse vectors and the wave partials of the sums share a place: 53 x 53 nodes in
    complex128 with 100 iterations (170,352 bytes apart), 67 x 67 in complex64 with 30 (164,928)."""
    from paper_2103_17081_amd.binding import Solver
    print("case: largest tiles", prec, cells, maxit, flush=True)
    n, k = 2 * cells, 0.3 * 2 * cells
    cuts = [0, cells, n]
    S = schwarz.Schwarz(schwarz.Problem(k, n, np.asarray(cuts), np.asarray(cuts)))
    tol = 1e-8 if prec == 64 else 1e-2
    with Solver(k, n_intervals=n, cuts_x=cuts, cuts_y=cuts, inner_precision=prec, inner_tol=tol, inner_maxit=maxit,
                outer_maxit=2) as gpu:
        assert int(gpu.layout[:, 2].max()) == cells + 1
        rng = np.random.default_rng(11)
        fs = [crandn(rng, s.geom.ndof) for s in S.subs]
        packed = pack(S, gpu, fs).astype(np.complex64 if prec == 32 else np.complex128)
        u, iters, flags = gpu.op_inner_solve(to_gpu(torch, packed))
        us = unpack(S, gpu, to_np(u).astype(np.complex128))
    for s, f, ug, it in zip(S.subs, fs, us, iters):
        d = s.defl
        ur, itr, _ = s.deflated_gmres(f, tol, maxit)
        print("iterations", int(it), itr, flush=True)
        assert abs(int(it) - itr) <= 1
        if prec == 32:
            assert np.linalg.norm(d.P(f - s.B @ ug)) <= 2 * tol * np.linalg.norm(d.P(f))
        elif it == itr:
            assert np.linalg.norm(ug - ur) <= 1e-8 * np.linalg.norm(ur)
