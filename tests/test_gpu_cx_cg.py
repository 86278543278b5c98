"""Conjugate gradients of the tVMC system at iteration limits around the interval of the host's readback (8):
none, one, just before, at and just after it, and a limit beyond convergence, against the same iterations in numpy
on the dense S; a zero force; a tolerance met between two readbacks.

What is compared is the residual: the recursive one that the solver reports stays within k x (condition of S + shift,
below 1e4 here) x 2^-52 x 10 of the true residual of the y it returns, 1e-9 for a dozen iterations.  (The iterates
of two orders of summation drift apart geometrically, so they are not compared.)
"""
import numpy as np
import pytest
import torch

from oracle.lattice import links_from_powers
from paper_2503_20566_amd import synth
from tests.test_gpu_tvmc import complex_theta, dense_O, handle

pytestmark = pytest.mark.gpu
SHIFT = 0.05


@pytest.fixture(scope="module")
def system(lib):
    L, N, Dk, B = 3, 2, 2, 48
    P, _, _ = handle(lib, L, N, Dk)
    theta = complex_theta(P.n_params, 11)
    powers = synth.plaquette_powers(B, L, N, seed=2)
    links = np.stack([links_from_powers(powers[b], N) for b in range(B)])
    th, lk = torch.from_numpy(theta).cuda(), torch.from_numpy(links).cuda()
    proj, bid, valid = P.cx_project(th, lk)
    ws = P.workspace(B, lib.PEPS_WS_TVMC)
    la, _ = P.cx_amplitude(proj, valid, ws)
    O = P.cx_logderiv(proj, valid, ws)
    el = P.cx_local_energy(th, lk, proj, valid, ws)
    D = dense_O(P, None, O.cpu().numpy(), bid.cpu().numpy())
    D = D - D.mean(0)
    e = el.cpu().numpy()
    S = D.conj().T @ D / B + SHIFT * np.eye(D.shape[1])
    g = D.conj().T @ (e - e.mean()) / B
    assert np.linalg.eigvalsh(S)[-1] / SHIFT < 1e4
    return P, (O, bid, valid, el, la, ws), S, g


def cg(S, g, k):
    y, r = np.zeros_like(g), g.copy()
    p, rr = r.copy(), np.vdot(r, r).real
    res = [rr]
    for _ in range(k):
        q = S @ p
        a = rr / np.vdot(p, q).real
        y, r = y + a * p, r - a * q
        new = np.vdot(r, r).real
        p, rr = r + new / rr * p, new
        res.append(rr)
    return y, res


def solve(P, args, e=None, **kw):
    O, bid, valid, el, la, ws = args
    out = P.tvmc_rhs(O, bid, valid, el if e is None else e, la, ws, shift=SHIFT, **kw)
    x = out[0].cpu().numpy()
    return (x if np.iscomplexobj(x) else x[..., 0] + 1j * x[..., 1]).reshape(-1), out


def check(P, args, S, g, expected, **kw):
    x, (_, _, its, rel) = solve(P, args, **kw)
    y = 1j * x  # alphadot = -i y
    assert its == expected
    assert abs(np.linalg.norm(g - S @ y) / np.linalg.norm(g) - rel) <= 1e-9
    return rel


@pytest.mark.parametrize("k", [0, 1, 7, 8, 9, 10])
def test_iteration_limits_around_the_readback(system, k):
    P, args, S, g = system
    rel = check(P, args, S, g, k, max_iter=k, rtol=0.0)
    assert (rel == 1.0) == (k == 0)


def test_tolerance_met_between_readbacks(system):
    P, args, S, g = system
    _, res = cg(S, g, 12)
    for k in (3, 8, 11):
        rtol = float(np.sqrt(res[k] / res[0]) * 1.01)
        first = next(i for i, r in enumerate(res) if r <= rtol ** 2 * res[0])
        assert check(P, args, S, g, first, max_iter=200, rtol=rtol) <= rtol


def test_zero_force_takes_no_iteration(system):
    P, args, S, g = system
    x, out = solve(P, args, e=torch.zeros_like(args[3]), max_iter=50, rtol=0.0)
    assert not x.any() and 0 in out[1:]
