"""An entry that a caller writes into a row's own column (a padding slot of the builder)
counts in the tiled recurrence as it does in the sweep of one step per launch, also
where every other entry has one value, which the tiled form then does not read.

Both forms form every value of T_n from the same operands in the same order: the kept
vectors are equal bit for bit, the moments differ by the order of N double sums (at
most about 2 eps sqrt(N) of mu_0 = N; held to 1e-13 N).
"""
import pytest
import torch

from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G
from tests.test_parity_tiles import STATE, _sweep_size

pytestmark = pytest.mark.gpu


def _run(H, a, b, r, M, prec, nbytes):
    work = torch.zeros(nbytes, dtype=torch.uint8, device=G.DEV)
    mu = tbkpm.kpm_moments(H, a, b, r, M, prec, work=work)
    return mu, work[STATE:STATE + H.n_rows * r.shape[1] * 3 * r.element_size()].clone()


@pytest.mark.parametrize("fmt,prec,nx,ny,R", [("sell_f32", "c32", 422, 420, 1), ("sell_f64", "f64", 70, 72, 2)])
def test_an_entry_in_its_own_column_counts(fmt, prec, nx, ny, R):
    s = synth.graphene_sheet(nx, ny, 0.0, 0)
    s.periodic = (1, 0, 0)                        # rows of two neighbours at the open edges
    H = G.build(s, fmt=fmt, slice=16)
    a, b = H.scale()
    a, M = 1.2 * a, 40
    r = tbkpm.random_phase(4, s.n, R, prec)
    t = H.tensors
    assert s.n % 16 == 0 and t["val"].numel() == 3 * s.n      # every slice is three wide
    pad = torch.nonzero(t["val"] == 0).flatten()
    k = int(pad[len(pad) // 2])
    row = 16 * (k // 48) + k % 16
    assert int(t["col"][k]) == row
    plain = tbkpm.kpm_moments(H, a, b, r, M, prec)
    t["val"][k] = 0.5
    tiled = _run(H, a, b, r, M, prec, tbkpm.workspace_size(H, R, M, prec))
    sweep = _run(H, a, b, r, M, prec, _sweep_size(H, R, M, prec))
    assert torch.equal(tiled[1], sweep[1])
    assert (tiled[0] - sweep[0]).abs().max().item() <= 1e-13 * s.n
    assert (tiled[0] - plain).abs().max().item() > 1e-3      # the entry moves mu_1 by about 0.5 / a
