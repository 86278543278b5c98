"""The row sweep and its adjoint at the edges of their instantiations (fused bonds up to 16, 32, 48, 72):
just below, at and just above each, with odd and even numbers of column pairs, against the oracle.
ln|Psi|, E_loc and every O element of two samples, without and with a stored tape (same bits).
Tolerances: those of the full-shape parity tests (ln|Psi| 1e-10 relative, E_loc 1e-9, O 1e-9 of the
largest element).
"""
import numpy as np
import pytest
import torch

from oracle.contract import amplitude
from oracle.energy import config_tables, local_energy
from oracle.layout import Layout, project
from oracle.logderiv import log_derivatives
from paper_2503_20566_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,chi", [(8, 7), (8, 8), (9, 9), (10, 15), (10, 17), (11, 23), (11, 24), (12, 25), (13, 35)])
@pytest.mark.parametrize("lanes", [8, 4])
def test_row_classes(lib, L, chi, lanes):
    N, Dk, B = 2, 2, 2
    print("row class", L, chi, lanes, flush=True)
    c, e = config_tables(N, 1.0, 0.4)
    lay = Layout(L, N, [Dk] * N)
    theta = synth.theta_normals(lay.n_params, N * Dk)
    powers = torch.from_numpy(synth.plaquette_powers(B, L, N, seed=100 * L + chi)).cuda()
    got = []
    for tape in (False, True):
        P = lib.Peps(L, N, Dk, chi, c, e, keep_tape=tape)
        t = P.get_tuning()
        t["jacobi_lanes"] = lanes
        P.set_tuning(t)
        links = P.links_from_powers(powers)
        th = torch.from_numpy(theta).cuda()
        proj, bid, valid = P.project(th, links)
        ws = P.workspace(B)
        la, sg = P.amplitude(proj, valid, ws)
        O, _ = P.logderiv(proj, bid, valid, ws)
        if not tape:
            P.amplitude(proj, valid, ws)
            el = P.local_energy(th, links, proj, valid, ws).cpu().numpy()
        got.append((la.cpu().numpy(), sg.cpu().numpy(), O.cpu().numpy()))
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    la, sg, O = got[0]
    lh = links.cpu().numpy()
    for b in range(B):
        ok, T, _ = project(lay, theta, lh[b])
        o_la, o_sg = amplitude(T, chi)
        assert ok and abs(la[b] - o_la) <= 1e-10 * abs(o_la) and sg[b] == o_sg
        o_el = local_energy(lay, theta, lh[b], chi, c, e)
        assert abs(el[b] - o_el) <= 1e-9 * max(1.0, abs(o_el)), (el[b], o_el)
        _, grads = log_derivatives(T, chi)
        scale = max(np.max(np.abs(g)) for row in grads for g in row)
        for y in range(L):
            for x in range(L):
                g = grads[y][x].reshape(-1)
                assert np.max(np.abs(O[b, y * L + x, :g.size] - g)) <= 1e-9 * scale
