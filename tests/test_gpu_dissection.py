"""Global coarse solve at the sizes and wave numbers where its solver changes, against the oracle's E_0.

Nested dissection: a grid that is one box (1 and 10 unknowns a side), the first that is cut (11),
unequal halves and depths (21, 23, 45); at 9 and at 7.9 coarse intervals per wavelength, the two
sides of the choice between it and the cyclic reduction; and k^2 next to an eigenvalue of a smallest box
(relative distance 1e-4 and 1e-8, which costs its pivots 4 and 8 digits: solves are refined, or
the handle goes back to the reduction).

Bound: the set-up refines above an estimated relative error of 3e-12 of the solution.  With three
times that for another vector than the estimate's, ||E_0 y - t|| <= 1e-11 ||E_0|| ||y||; the
cyclic reduction's bound is that of the other coarse tests, 1e-7 ||t||.
"""

import numpy as np
import pytest
import scipy.linalg as sl
import scipy.sparse as sp

from oracle import coarse_space, fem
from tests.gpu_common import crandn, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def _coarse(k, n, m):
    z = coarse_space.z2d(n, m)
    return sp.csr_matrix((z.T @ fem.helmholtz_matrix(k, n) @ z).real)


def _solve(torch, k, n, m, rng):
    from paper_2103_17081_amd.binding import Solver
    with Solver(k, n_intervals=n, cuts_x=[0, n // 2, n], cuts_y=[0, n // 2, n], coarse_intervals=m,
                outer_maxit=2) as s:
        t = crandn(rng, (m - 1) ** 2)
        return t, to_np(s.op_global_coarse_solve(to_gpu(torch, t)))


@pytest.mark.parametrize("per_wave", [9.0, 7.9])
@pytest.mark.parametrize("m", [2, 11, 12, 22, 24, 46])
def test_coarse_solve_sizes(torch, m, per_wave):
    k, n = 2 * np.pi * m / per_wave, 2 * m
    t, y = _solve(torch, k, n, m, np.random.default_rng(m))
    E = _coarse(k, n, m)
    r = np.linalg.norm(E @ y - t)
    if per_wave >= 8.0:
        assert r <= 1e-11 * abs(E).sum(axis=1).max() * np.linalg.norm(y)
    else:
        assert r <= 1e-7 * np.linalg.norm(t)


@pytest.mark.parametrize("off", [1e-4, 1e-8])
def test_coarse_solve_next_to_a_box_resonance(torch, off):
    m, n = 46, 92
    box = [y * (m - 1) + x for y in range(12, 22) for x in range(12, 22)]   # a smallest box: 10 x 10
    E0 = _coarse(0.0, n, m)[box][:, box].toarray()
    E1 = E0 - _coarse(1.0, n, m)[box][:, box].toarray()
    mu = sl.eigvals(E0, E1)
    mu = np.sort(mu[abs(mu.imag) < 1e-9 * abs(mu.real)].real)
    k = float(np.sqrt(mu[mu > 0][0] * (1 + off)))
    assert 2 * np.pi * m / k >= 8.0
    t, y = _solve(torch, k, n, m, np.random.default_rng(5))
    E = _coarse(k, n, m)
    assert np.linalg.norm(E @ y - t) <= 1e-11 * abs(E).sum(axis=1).max() * np.linalg.norm(y)
