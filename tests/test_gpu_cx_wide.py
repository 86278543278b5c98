"""The complex contraction on both sides of its size rule: working states in LDS (6 x 6 at D_k = 3, 10 x 10 at
D_k = 2 are the largest) and in global memory (7 x 7 and 11 x 11 the smallest there; 8 x 8 for an odd and an even
number of sites before the tail), for batches whose row pairs are split over the workgroups and not.

Tensors near 1 make every amplitude a sum without cancellation, so that a contraction of L^2 sites, each a sum of
D_k^2 products, is within 10 eps L^2 D_k^2 of the exact one:
* sum_k T_k O_k = 1 for every site (the environments against the amplitude);
* E_loc against the amplitudes of the flipped configurations;
* a workspace without the split's slots gives the same E_loc and O.
"""
import numpy as np
import pytest
import torch

from oracle.energy import config_tables
from oracle.lattice import links_from_powers
from paper_2503_20566_amd import synth

pytestmark = pytest.mark.gpu


def flipped(links, x, y, t, N):
    """Links with plaquette (x, y) lowered by P^-t: h(x,y), v(x+1,y) - t; h(x,y+1), v(x,y) + t."""
    out = links.copy()
    for d, i, j, s in ((0, y, x, -t), (1, y, x + 1, -t), (0, y + 1, x, t), (1, y, x, t)):
        out[:, d, i, j] = (out[:, d, i, j].astype(int) + s) % N
    return out


@pytest.mark.parametrize("c64", [False, True])
@pytest.mark.parametrize("L,N,Dk,B", [(6, 2, 3, 3), (7, 2, 3, 3), (8, 2, 3, 2), (10, 2, 2, 3), (11, 2, 2, 2), (4, 3, 2, 5)])
def test_cx_states_in_lds_and_in_memory(lib, L, N, Dk, B, c64):
    c, e = config_tables(N, 1.0, 0.4)
    P = lib.Peps(L, N, Dk, 4, c, e, dtype=lib.PEPS_C64_EXACT if c64 else lib.PEPS_C128_EXACT)
    rng = np.random.Generator(np.random.PCG64(L * 10 + Dk))
    theta = 1 + 0.3 * (rng.standard_normal(P.n_params) + 1j * rng.standard_normal(P.n_params))
    th = torch.from_numpy(theta).cuda()
    powers = synth.plaquette_powers(B, L, N, seed=5)
    links = np.stack([links_from_powers(powers[b], N) for b in range(B)])
    tol = 10 * (2.0 ** -23 if c64 else 2.0 ** -52) * L * L * Dk * Dk

    def amplitudes(lk):
        proj, _, valid = P.cx_project(th, torch.from_numpy(lk).cuda())
        la, ph = P.cx_amplitude(proj, valid, P.workspace(lk.shape[0], lib.PEPS_WS_AMPLITUDE))
        return la.cpu().numpy(), ph.cpu().numpy().reshape(lk.shape[0], -1)

    lk = torch.from_numpy(links).cuda()
    proj, bid, valid = P.cx_project(th, lk)
    assert valid.all()
    S, W = Dk ** L, Dk ** (L + 1)
    up = lambda n: (n + 255) // 256 * 256
    cb = 8 if c64 else 16
    small = up(cb * B * 2 * (L + 1) * S) + up(8 * B * 2 * (L + 1)) + up(cb * B * L * W)
    small += up(cb * B * 2 * W) if W > 2187 else 0
    full = P.workspace_bytes(B, lib.PEPS_WS_AMPLITUDE)
    assert full > small
    res = []
    for nbytes in (full, small):
        ws = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
        P.cx_amplitude(proj, valid, ws)
        O = P.cx_logderiv(proj, valid, ws)
        E = P.cx_local_energy(th, lk, proj, valid, ws)
        res.append((torch.view_as_complex(O.reshape(O.shape[:3] + (2,))) if not O.is_complex() else O,
                    torch.view_as_complex(E.reshape(B, 2)) if not E.is_complex() else E))
    O, E = (r.cpu().numpy() for r in res[0])
    # the split changes the order of a few FP64 sums only
    assert np.abs(res[1][0].cpu().numpy() - O).max() <= 1e-12 * np.abs(O).max()
    assert np.abs(res[1][1].cpu().numpy() - E).max() <= 1e-12 * np.abs(E).max()
    T = proj.cpu().numpy()
    T = (T if np.iscomplexobj(T) else T[..., 0::2] + 1j * T[..., 1::2] if T.ndim == 3 else T[..., 0] + 1j * T[..., 1])
    euler = (T.reshape(O.shape) * O).sum(-1)
    assert np.abs(euler - 1).max() <= tol
    la, ph = amplitudes(links)
    psi = lambda p: p[:, 0] if np.iscomplexobj(p) else p[:, 0] + 1j * p[:, 1]
    ref = np.asarray(e)[links[:, 0, :, : L - 1].astype(int)].sum((1, 2)).astype(complex)
    ref += np.asarray(e)[links[:, 1, : L - 1, :].astype(int)].sum((1, 2))
    scale = np.abs(ref)
    for y in range(L - 1):
        for x in range(L - 1):
            for t in range(1, N):
                if c[t] == 0:
                    continue
                l2, p2 = amplitudes(flipped(links, x, y, t, N))
                r = c[t] * np.exp(l2 - la) * psi(p2) / psi(ph)
                ref += r
                scale += np.abs(r)
    assert np.abs(E - ref).max() <= (2 * tol * scale).max()
