"""kpm_last_form names the form of the recurrence that ran."""
import numpy as np
import pytest
import torch

from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G

pytestmark = pytest.mark.gpu
M = 50


def _single(nx, ny, R=2, shuffle=False, work=False):
    s = synth.graphene_sheet(nx, ny, 0.05, 1)
    if shuffle:
        p = np.random.default_rng(1).permutation(s.n)
        s.pos, s.species = s.pos[p].copy(), s.species[p].copy()
    H = G.build(s, fmt="sell_f32", slice=64, reorder=not shuffle)
    a, b = H.scale()
    r = tbkpm.random_phase(3, s.n, R)
    w = torch.empty(tbkpm.least_workspace_size(H, R, M, "c32"), dtype=torch.uint8, device=G.DEV) if work else None
    tbkpm.kpm_moments(H, a, b, r, M, work=w)
    return tbkpm.last_form()


def test_single_runs():
    tiles, steps = _single(110, 100)
    assert tiles > 100 and 2 <= steps <= 16
    assert _single(20, 30) == (1, M - 1)
    assert _single(110, 100, work=True) == (0, 1)           # the sweep's workspace
    assert _single(100, 90, shuffle=True) == (0, 1)         # rows far from their neighbours


def test_stacks_and_the_persistent_launch():
    snaps = [synth.graphene_sheet(40 + k, 50, 0.05, k) for k in range(3)]
    pos, sp, seg, boxes = synth.stack(snaps)
    H = tbkpm.build_hamiltonian_batched(G.to_dev(pos), G.to_dev(sp), seg, boxes, (1, 1, 0), [0.0], [[-2.7]])
    a, b = H.scales()
    r = tbkpm.random_phase(2, int(seg[-1]), 2)
    tbkpm.kpm_moments_batched(H, a, b, r, M)
    assert tbkpm.last_form()[0] >= 3
    tbkpm.kpm_moments_batched(H, a, b, r, M, config=tbkpm.make_config(1, 1, 1, 0, 1, 1))
    assert tbkpm.last_form() == (0, M - 1)
