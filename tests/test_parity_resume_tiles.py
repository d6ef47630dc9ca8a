"""Resume on matrices of several tiles: a run split at any moment gives, bit for bit, the
moments of the one-shot run, before and after the split.

The moments are sums per tile, so where the tiles end must not depend on the number of
moments of the call: sheets of which some tiles are cut to fit their halos, rows of 3 to
6 entries.
"""
import pytest
import torch

from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,sigma", [(100, 100, 0.05), (260, 130, 0.05), (130, 300, 0.09), (190, 120, 0.16),
                                         (150, 40, 0.0)])
@pytest.mark.parametrize("fmt,prec,R", [("sell_f32", "c32", 1), ("sell_f32", "c32", 3), ("sell_f64", "f64", 2)])
def test_split_runs_add_up_to_the_one_shot_run(nx, ny, sigma, fmt, prec, R):
    s = synth.graphene_sheet(nx, ny, sigma, 3)
    H = G.build(s, fmt=fmt, slice=32)
    a, b = H.scale()
    r = tbkpm.random_phase(2, s.n, R, prec)
    M = 400
    one = tbkpm.kpm_moments(H, a, b, r, M, prec)
    for stops in ((150,), (2, 9, 201), (200, 202)):
        work = tbkpm.alloc_workspace(H, R, M, prec)
        k0 = 0
        for k1 in stops + (M,):
            mu = torch.empty((R, k1), dtype=torch.float64, device=G.DEV)
            tbkpm.kpm_moments(H, a, b, r if k0 == 0 else None, k1, prec, work=work, mu=mu, n_start=k0, R=R)
            assert torch.equal(mu[:, k0:], one[:, k0:k1]), (k0, k1)
            k0 = k1
