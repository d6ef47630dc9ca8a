"""Runs whose planes would take more than 32 GB go through their vectors in sets
(14 M rows, 33 vectors in FP64: three sets of 16 and one of padding alone): vectors bit
for bit those of the sweep of one step per launch, moments to the order of N double sums
(1e-13 N), a split run bit for bit the one-shot run.
"""
import pytest
import torch

from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G
from tests.test_parity_tiles import STATE, _sweep_size

pytestmark = pytest.mark.gpu
NX, NY, R = 1850, 1900, 33
PREC = "f64"


@pytest.fixture(scope="module")
def system():
    s = synth.graphene_sheet(NX, NY, 0.04, 2)
    H = G.build(s, fmt="sell_f64", slice=64)
    r = tbkpm.random_phase(1, s.n, R, PREC)
    yield s.n, H, r
    del H, r
    torch.cuda.empty_cache()


def test_sets_of_vectors_equal_the_sweep(system):
    n, H, r = system
    a, b = H.scale()
    M = 12
    full, small = tbkpm.workspace_size(H, R, M, PREC), _sweep_size(H, R, M, PREC)
    vec = n * 64 * 16
    assert full - small < 5 * (n * 16 * 16) + 200 * n        # planes of 16 vectors (all 33: more than twice that)
    works = [torch.zeros(k, dtype=torch.uint8, device=G.DEV) for k in (full, small)]
    mus = [tbkpm.kpm_moments(H, a, b, r, M, PREC, work=w) for w in works]
    assert (mus[0] - mus[1]).abs().max().item() <= 1e-13 * n
    for k in range(3):
        at = STATE + k * vec
        assert torch.equal(works[0][at:at + vec], works[1][at:at + vec]), k
    del works[1:]
    torch.cuda.empty_cache()
    # split: 5 moments, then the rest
    first = torch.empty((R, 5), dtype=torch.float64, device=G.DEV)
    rest = torch.empty((R, M), dtype=torch.float64, device=G.DEV)
    tbkpm.kpm_moments(H, a, b, r, 5, PREC, work=works[0], mu=first)
    tbkpm.kpm_moments(H, a, b, None, M, PREC, work=works[0], mu=rest, n_start=5, R=R)
    assert torch.equal(torch.cat([first, rest[:, 5:]], 1), mus[0])


def test_sets_of_vectors_in_the_doubling_form(system):
    n, H, r = system
    a, b = H.scale()
    M = 24
    cfg = tbkpm.with_doubling(tbkpm.default_config(H, R, PREC), 1)
    mus = []
    for nbytes in (tbkpm.workspace_size(H, R, M, PREC, cfg), _sweep_size(H, R, M, PREC, doubling=1)):
        work = torch.zeros(nbytes, dtype=torch.uint8, device=G.DEV)
        tbkpm.step_timer(True)
        mus.append(tbkpm.kpm_moments(H, a, b, r, M, PREC, work=work, config=cfg))
        assert tbkpm.step_timer_read()[1] == M // 2
        tbkpm.step_timer(False)
        del work
        torch.cuda.empty_cache()
    assert (mus[0] - mus[1]).abs().max().item() <= 1e-13 * n
