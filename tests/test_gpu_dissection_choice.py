"""Which solver a two-level handle takes for its coarse grid, told by the bytes of a solve (dd_stats.coarse_bytes): nested
dissection, dissection with every solve refined, or the block cyclic reduction.

At 9 intervals per wavelength the dissection, at 7.9 the reduction.  With k^2 next to an eigenvalue of a smallest box
(relative distance 1e-2, 1e-4, 1e-8) its pivots lose 2, 4 and 8 digits, and the set-up's error estimate, which grows with
the square of what they lose, lies below the 3e-12 above which solves are refined, between that and 1e-6, and above
1e-6, where the reduction takes over.

Bound of the solutions: ||E_0 y - t|| <= 1e-11 ||E_0|| ||y||, as in the other test of this solver."""

import numpy as np
import pytest
import scipy.linalg as sl

from tests.gpu_common import crandn, to_gpu, to_np
from tests.test_gpu_dissection import _coarse

pytestmark = pytest.mark.gpu

M, N = 46, 92


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def _bytes(torch, k):
    """Bytes of a coarse solve on a handle of wave number k, after checking one against E_0."""
    from paper_2103_17081_amd.binding import Solver
    rng = np.random.default_rng(5)
    with Solver(k, n_intervals=N, cuts_x=[0, N // 2, N], cuts_y=[0, N // 2, N], coarse_intervals=M, outer_maxit=1) as s:
        t = crandn(rng, (M - 1) ** 2)
        y = to_np(s.op_global_coarse_solve(to_gpu(torch, t)))
        _, st = s.solve(to_gpu(torch, crandn(rng, (N - 1) ** 2)), check=False)
    E = _coarse(k, N, M)
    assert np.linalg.norm(E @ y - t) <= 1e-11 * abs(E).sum(axis=1).max() * np.linalg.norm(y)
    return st["coarse_bytes"]


def test_choice(torch):
    plain, reduction = _bytes(torch, 2 * np.pi * M / 9.0), _bytes(torch, 2 * np.pi * M / 7.9)
    refined = 2 * plain + (M - 1) ** 2 * (9 * 8 + 6 * 16)   # two sweeps, a residual and an addition
    assert len({plain, reduction, refined}) == 3
    box = [y * (M - 1) + x for y in range(12, 22) for x in range(12, 22)]   # a smallest box: 10 x 10
    E0 = _coarse(0.0, N, M)[box][:, box].toarray()
    mu = sl.eigvals(E0, E0 - _coarse(1.0, N, M)[box][:, box].toarray())
    mu = np.sort(mu[abs(mu.imag) < 1e-9 * abs(mu.real)].real)
    for off, want in ((1e-2, plain), (1e-4, refined), (1e-8, reduction), (0.0, reduction)):
        print("case: distance", off, flush=True)
        assert _bytes(torch, float(np.sqrt(mu[mu > 0][0] * (1 + off)))) == want
