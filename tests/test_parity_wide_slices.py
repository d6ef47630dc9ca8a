"""Slices stored wider than the largest row degree the Hamiltonian states (its padding is
the caller's affair): rows are read as wide as `ptr` says, whatever the size.

The reference is the same Hamiltonian with its widest slice stated.  Vectors are equal bit
for bit, moments differ by the order of N double sums: held to 1e-13 N.
"""
import pytest
import torch

from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(12, 10), (20, 30), (90, 80)])          # one tile, one tile, several
@pytest.mark.parametrize("fmt,prec,R", [("sell_f32", "c32", 3), ("sell_f64", "f64", 1)])
def test_slices_wider_than_the_stated_degree(nx, ny, fmt, prec, R):
    s = synth.graphene_sheet(nx, ny, 0.14, 7)
    H = G.build(s, fmt=fmt, slice=16)
    assert H.st.max_degree > 3
    a, b = H.scale()
    r = tbkpm.random_phase(8, s.n, R, prec)
    M = 30
    want = tbkpm.kpm_moments(H, a, b, r, M, prec)
    vx = tbkpm.build_velocity(H, G.to_dev(s.pos), s.box, s.periodic, 0)
    want_nu = tbkpm.vac_moments(H, vx, a, b, r, M, 3, 0.1, precision=prec)
    work = tbkpm.alloc_workspace(H, R, M, prec)
    H.st.max_degree = 3
    for seeded in (False, True):
        got = (tbkpm.kpm_moments_seeded(H, a, b, 8, R, M, prec) if seeded
               else tbkpm.kpm_moments(H, a, b, r, M, prec))
        assert (got - want).abs().max().item() <= 1e-13 * s.n
    first = torch.empty((R, 11), dtype=torch.float64, device=G.DEV)
    rest = torch.empty((R, M), dtype=torch.float64, device=G.DEV)
    tbkpm.kpm_moments(H, a, b, r, 11, prec, work=work, mu=first)
    tbkpm.kpm_moments(H, a, b, None, M, prec, work=work, mu=rest, n_start=11, R=R)
    assert (torch.cat([first, rest[:, 11:]], 1) - want).abs().max().item() <= 1e-13 * s.n
    nu = tbkpm.vac_moments(H, vx, a, b, r, M, 3, 0.1, precision=prec)
    assert (nu - want_nu).abs().max().item() <= 1e-13 * max(want_nu.abs().max().item(), s.n)
    tbkpm.step_timer(True)
    try:
        got = tbkpm.kpm_moments(H, a, b, r, M, prec)
        assert tbkpm.step_timer_read()[1] == M - 1
    finally:
        tbkpm.step_timer(False)
    assert (got - want).abs().max().item() <= 1e-13 * s.n
