"""Stacks and doubling runs of so few moments that listing tiles would cost more than the
steps: the sweep runs (its workspace is all they ask for), with the moments that longer
calls give (the order of N double sums apart: 1e-13 N)."""
import pytest
import torch

from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,R", [(((20, 25),), 2), (((20, 25), (70, 60)), 3), (((150, 150), (130, 140)), 8)])
def test_stacks_of_few_moments(dims, R):
    snaps = [synth.graphene_sheet(nx, ny, 0.05, k) for k, (nx, ny) in enumerate(dims)]
    pos, sp, seg, boxes = synth.stack(snaps)
    H = tbkpm.build_hamiltonian_batched(G.to_dev(pos), G.to_dev(sp), seg, boxes, (1, 1, 0), [0.0], [[-2.7]])
    a, b = H.scales()
    r = tbkpm.random_phase(2, int(seg[-1]), R)
    want = tbkpm.kpm_moments_batched(H, a, b, r, 60)
    tiles = []
    for M in (2, 3, 5, 11, 28, 29, 60):
        tiles.append(tbkpm.workspace_size_batched(H, R, M, "c32") > tbkpm.least_workspace_size_batched(H, R, M, "c32"))
        got = tbkpm.kpm_moments_batched(H, a, b, r, M)
        assert (got - want[:, :, :M]).abs().max().item() <= 1e-13 * int(seg[-1])
    assert not tiles[0] and tiles[-1] and tiles == sorted(tiles)


@pytest.mark.parametrize("nx,ny,R", [(20, 25, 2), (70, 60, 3), (150, 150, 8)])
def test_doubling_of_few_moments(nx, ny, R):
    s = synth.graphene_sheet(nx, ny, 0.05, 4)
    H = G.build(s, fmt="sell_f64", slice=32)
    a, b = H.scale()
    r = tbkpm.random_phase(2, s.n, R, "f64")
    cfg = tbkpm.with_doubling(tbkpm.default_config(H, R, "f64"), 1)
    want = tbkpm.kpm_moments(H, a, b, r, 60, "f64", config=cfg)
    tiles = []
    for M in (2, 3, 7, 8, 19, 20, 60):
        tiles.append(tbkpm.workspace_size(H, R, M, "f64", cfg) > tbkpm.least_workspace_size(H, R, M, "f64", cfg))
        got = tbkpm.kpm_moments(H, a, b, r, M, "f64", config=cfg)
        assert (got - want[:, :M]).abs().max().item() <= 1e-13 * s.n
    assert not tiles[0] and tiles[-1] and tiles == sorted(tiles)


def test_a_run_that_can_be_continued_takes_tiles_however_short():
    H = G.build(synth.graphene_sheet(70, 60, 0.05, 4), fmt="sell_f32", slice=32)
    assert tbkpm.workspace_size(H, 3, 2, "c32") > tbkpm.least_workspace_size(H, 3, 2, "c32")
