"""The per-block sums of the SR build and of the vjp (k_sr_blocks) against a plain scatter in float64 on
the CPU, at the sizes where their chunks, wave shares and lane groups change: batches around 64 and
1024 samples (a ballot, a staged chunk), sites with few and with more than 16 blocks, Dk = 1 and 2,
both occupations' blocks of a matter problem, and batches with invalid samples.

Tolerance: a sum of B terms in any order differs from another by at most B eps times the sum of the
terms' magnitudes; the covariances add three such sums, and the factors of the products one eps each.
"""
import numpy as np
import pytest
import torch

from paper_2503_20566_amd import synth

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


def scatter(P, bid, rows):
    """Dense [B, n_params] of block-sparse rows [B, L*L, P4]."""
    B = rows.shape[0]
    out = np.zeros((B, P.n_params))
    L = P.L
    for s in range(L * L):
        x, y = s % L, s // L
        size = P.Dk ** (int(x > 0) + int(x < L - 1) + int(y > 0) + int(y < L - 1))
        at = P.site_offset[s] + bid[:, s].astype(np.int64)[:, None] * size + np.arange(size)[None, :]
        ok = bid[:, s] >= 0
        out[np.arange(B)[ok, None], at[ok]] = rows[ok, s, :size]
    return out


@pytest.mark.parametrize("L,N,Dk,matter,B,bad", [
    (3, 2, 1, False, 1, 0), (3, 2, 2, False, 63, 1), (4, 3, 2, False, 64, 0), (3, 3, 2, True, 65, 2),
    (4, 2, 2, False, 1023, 5), (3, 4, 2, False, 1024, 0), (3, 3, 2, False, 1025, 1), (3, 8, 1, False, 2100, 7),
])
def test_sr_sums_and_matvec(lib, L, N, Dk, matter, B, bad):
    P = lib.Peps(L, N, Dk, 4, [0.0] + [-1.0] * (N - 1), [0.1] * N, matter=matter)
    powers = torch.from_numpy(synth.plaquette_powers(B, L, N)).cuda()
    if matter:
        links = P.matter_links(powers, torch.from_numpy(synth.occupations(B, L, N)).cuda())
    else:
        links = P.links_from_powers(powers)
    links[:bad, 0, 0, 0] = (links[:bad, 0, 0, 0] + 1) % N      # breaks the Gauss law of vertex (0, 0)
    theta = torch.from_numpy(synth.theta_normals(P.n_params, N * Dk)).cuda()
    _, bid, valid = P.project(theta, links)
    v = valid.cpu().numpy().astype(bool)
    assert v.sum() == B - bad
    rows = synth.normals((B, L * L, P.P4), 3)
    e, x = synth.normals((B,), 4), synth.normals((P.n_params,), 5)
    ws = P.workspace(B, lib.PEPS_WS_LOGDERIV)
    up = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    F, om, Sv = (t.cpu().numpy() for t in P.sr_build(up(rows), bid, valid, up(e), ws, v=up(x)))
    A = scatter(P, bid.cpu().numpy(), rows)[v]
    n = len(A)
    mean = A.mean(0) if n else np.zeros(P.n_params)
    mag = np.abs(A).sum(0) / max(n, 1)
    tol = 8 * (B + P.n_params) * EPS
    assert np.all(np.abs(om - mean) <= tol * mag)
    ref = A.T @ e[v] / n - mean * e[v].mean()
    bound = np.abs(A).T @ np.abs(e[v]) / n + mag * np.abs(e[v]).mean()
    assert np.all(np.abs(F - ref) <= tol * bound)
    ov = A @ x
    ref = A.T @ ov / n - mean * ov.mean()
    mov = np.abs(A) @ np.abs(x)
    assert np.all(np.abs(Sv - ref) <= tol * (np.abs(A).T @ mov / n + mag * mov.mean()))


@pytest.mark.parametrize("B,weights", [(1, True), (130, False), (1030, True)])
def test_vjp_is_the_weighted_sum_of_O(lib, B, weights):
    L, N, Dk = 3, 3, 2
    P = lib.Peps(L, N, Dk, 4, [0.0, -1.0, -1.0], [0.1] * N)
    links = P.links_from_powers(torch.from_numpy(synth.plaquette_powers(B, L, N)).cuda())
    theta = torch.from_numpy(synth.theta_normals(P.n_params, N * Dk)).cuda()
    proj, bid, valid = P.project(theta, links)
    ws = P.workspace(B)
    P.amplitude(proj, valid, ws)
    w = synth.normals((B,), 6)
    O, vjp = P.logderiv(proj, bid, valid, ws, w=torch.from_numpy(w).cuda() if weights else None, want_vjp=True)
    A = scatter(P, bid.cpu().numpy(), O.cpu().numpy())
    w = w if weights else np.ones(B)
    assert np.all(np.abs(vjp.cpu().numpy() - A.T @ w) <= 8 * B * EPS * (np.abs(A).T @ np.abs(w)))
