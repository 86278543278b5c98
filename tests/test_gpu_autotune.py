"""What the autotuner reports is what the kernels run: small_waves chooses no kernel, so one time stands for both of
its values (fused bonds up to 32), and the kernels of fused bonds above 72 run eight Jacobi lanes.
"""
import pytest
import torch

from oracle.energy import config_tables
from paper_2503_20566_amd import synth

pytestmark = pytest.mark.gpu


def tuned(lib, L, N, chi, B):
    c, e = config_tables(N, 1.0, 0.4)
    P = lib.Peps(L, N, 2, chi, c, e)
    th = torch.from_numpy(synth.theta_normals(P.n_params, N * 2)).cuda()
    links = P.links_from_powers(torch.from_numpy(synth.plaquette_powers(B, L, N)).cuda())
    proj, _, valid = P.project(th, links)
    before = P.get_tuning()
    r = P.autotune(proj, valid, P.workspace(B, lib.PEPS_WS_AMPLITUDE | lib.PEPS_WS_ENERGY))
    assert P.get_tuning() == r["tuning"]
    return before, r["tuning"], r["candidates"]


@pytest.mark.parametrize("chi", [4, 16])
def test_one_time_for_both_wave_counts(lib, chi):
    before, best, found = tuned(lib, 8, 2, chi, 16)
    assert len(found) == 40 and best["small_waves"] == before["small_waves"]
    key = lambda c: tuple(c[f] for f in ("jacobi_lanes", "precond", "precond_min", "up"))
    for waves in (2, 4):
        assert len({key(c) for c in found if c["small_waves"] == waves}) == 20
    times = {w: {key(c): c["ms"] for c in found if c["small_waves"] == w} for w in (2, 4)}
    assert times[2] == times[4] and min(times[2].values()) > 0.0
    # the choice is the fastest combination of those times
    total = {(a, b): min(t for k, t in times[2].items() if k[0] == a and k[2] == b and k[3] == 0)
             + min(t for k, t in times[2].items() if k[0] == a and k[2] == b and k[3] == 1) for a in (8, 4) for b in (16, 32)}
    assert total[best["jacobi_lanes"], best["precond_min"]] == min(total.values())


def test_large_bonds_report_eight_lanes(lib):
    _, best, found = tuned(lib, 12, 2, 40, 2)
    assert len(found) == 10 and best["jacobi_lanes"] == 8
    assert {c["jacobi_lanes"] for c in found} == {8} and {c["precond_min"] for c in found} == {16, 32}
