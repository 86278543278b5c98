"""How the conjugate gradients of sr_solve and tvmc_rhs end other than by their tolerance: a zero force, and a
breakdown (p.S p = 0) at the first iteration and at the second, between two readbacks of the complex solver.

Every number is exact.  Four samples give two parameters of one block a diagonal S: O = +-1 of parameter 0 in samples
0 and 1, O = +-2^-540 of parameter 1 in samples 2 and 3, so S = diag(1/2, 0): the second entry, 2^-1081, is below the
smallest number.  E = +-2 e_0 and +-2^541 e_1 make the force (e_0, e_1), with <O> = <E> = 0.  From (1, 1): q = (1/2, 0),
alpha = 2 / (1/2) = 4, x = (4, 4), r = (-1, 1), beta = 1, p = (0, 2), and S p = 0 ends it after one iteration with r.r
what it was.

The complex solver reads its state back after 8 iterations, after 2 at a tolerance of at least 1e-2, and then every 8:
tolerances of either kind, met at, before and after the first readbacks.
"""
import numpy as np
import pytest
import torch

from oracle.energy import config_tables
from tests.test_gpu_cx_cg import cg, check, system  # noqa: F401  (system: the fixture)

pytestmark = pytest.mark.gpu


def problem(lib, cplx, e0, e1):
    L, N, Dk, B = 3, 2, 2, 4
    c, e = config_tables(N, 1.0, 0.4)
    P = lib.Peps(L, N, Dk, 4, c, e, dtype=lib.PEPS_C128_EXACT if cplx else lib.PEPS_F64)
    O = np.zeros((B, L * L, Dk ** 4), dtype=np.complex128 if cplx else np.float64)
    O[0, 0, 0], O[1, 0, 0] = 1.0, -1.0
    O[2, 0, 1], O[3, 0, 1] = 2.0 ** -540, -(2.0 ** -540)
    E = np.array([2.0 * e0, -2.0 * e0, 2.0 ** 541 * e1, -(2.0 ** 541) * e1], dtype=O.dtype)
    dev = lambda a: torch.from_numpy(a).cuda()
    return P, dev(O), dev(np.zeros((B, L * L), dtype=np.int32)), dev(np.ones(B, dtype=np.uint8)), dev(E)


def solve(lib, cplx, e0, e1, max_iter):
    P, O, bid, valid, E = problem(lib, cplx, e0, e1)
    if cplx:
        la = torch.zeros(4, dtype=torch.float64, device="cuda")
        x, energy, its, rel = P.tvmc_rhs(O, bid, valid, E, la, P.workspace(4, lib.PEPS_WS_TVMC), shift=0.0,
                                         max_iter=max_iter, rtol=0.0)
        assert energy == 0.0
        return 1j * x.cpu().numpy(), its, rel            # alphadot = -i y
    x, F, mean, its, rel = P.sr_solve(O, bid, valid, E, P.workspace(4, lib.PEPS_WS_LOGDERIV), 0.0, max_iter, 0.0)
    F = F.cpu().numpy()
    assert not mean.any() and F[0] == e0 and F[1] == e1 and not F[2:].any()
    return x.cpu().numpy(), its, rel


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("e0,e1,max_iter,its,rel,x0,x1", [
    (1.0, 1.0, 50, 1, 1.0, 4.0, 4.0),    # breakdown at the second iteration
    (1.0, 1.0, 1, 1, 1.0, 4.0, 4.0),     # the limit just before it
    (0.0, 1.0, 50, 0, 1.0, 0.0, 0.0),    # breakdown at the first
    (1.0, 0.0, 50, 1, 0.0, 2.0, 0.0),    # solved by the first
    (0.0, 0.0, 50, 0, 0.0, 0.0, 0.0),    # no force
])
def test_ends(lib, cplx, e0, e1, max_iter, its, rel, x0, x1):
    x, got_its, got_rel = solve(lib, cplx, e0, e1, max_iter)
    assert (got_its, got_rel) == (its, rel)
    assert x[0] == x0 and x[1] == x1 and not x[2:].any()


@pytest.mark.parametrize("rtol", [0.5, 0.1, 1e-2, 0.99e-2, 1e-3, 1e-5])
@pytest.mark.parametrize("limit", [1, 2, 3, 200])
def test_tolerances_around_the_readbacks(system, rtol, limit):  # noqa: F811
    P, args, S, g = system
    _, res = cg(S, g, 40)
    met = next(i for i, r in enumerate(res) if r <= rtol ** 2 * res[0])
    assert all(abs(r / (rtol ** 2 * res[0]) - 1) > 1e-6 for r in res), "a residual too close to the bound to tell"
    rel = check(P, args, S, g, min(met, limit), max_iter=limit, rtol=rtol)
    assert (rel <= rtol) == (met <= limit)
