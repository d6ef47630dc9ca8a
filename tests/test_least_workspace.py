"""Where the device has no room for the workspace of the steps on tiles, the binding takes
the sweep's (one step per launch), as large as it was before tiles: every call that fitted
then still runs.  Moments differ by the order of N double sums: held to 1e-13 N."""
import pytest
import torch

from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G
from tests.test_parity_tiles import _sweep_size


def test_least_sizes_without_gpu():
    """Never above the full size, and equal to it where tiles are not offered."""
    for degree, tiles in ((3, True), (6, True), (7, False)):
        st = tbkpm.HamStruct(fmt=2, slice=64, n_rows=100000, n_entries=100032 * degree, max_degree=degree, n_seg=1,
                             n_orb=1)
        H = tbkpm.Hamiltonian(st, {}, None)
        for R in (1, 5):
            full, least = (f(H, R, 300, "c32") for f in (tbkpm.workspace_size, tbkpm.least_workspace_size))
            assert 3 * 100000 * R * 8 < least <= full and (least < full) == tiles
            full, least = (tbkpm.vac_workspace_size(H, R, 100, "c32", least=k) for k in (False, True))
            assert least <= full and (least < full) == tiles


@pytest.fixture
def room():
    """room(nbytes): from now on torch finds room for nbytes more."""
    def limit(nbytes):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        total = torch.cuda.get_device_properties(0).total_memory
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + nbytes) / total)
    yield limit
    torch.cuda.set_per_process_memory_fraction(1.0)


@pytest.mark.gpu
def test_binding_falls_back_to_the_least_workspace(room):
    s = synth.graphene_sheet(500, 400, 0.05, 2)
    M, R, spare = 12, 8, 96 << 20
    H = G.build(s, fmt="sell_f32", slice=64)
    a, b = H.scale()
    r = tbkpm.random_phase(3, s.n, R)
    assert tbkpm.least_workspace_size(H, R, M, "c32") == _sweep_size(H, R, M, "c32")
    want = tbkpm.kpm_moments(H, a, b, r, M)
    HB = tbkpm.build_hamiltonian_batched(G.to_dev(s.pos), G.to_dev(s.species), [0, s.n], [s.box], s.periodic, s.onsite,
                                         s.t_pair)
    wantB = tbkpm.kpm_moments_batched(HB, [a], [b], r, M)
    vx = tbkpm.build_velocity(H, G.to_dev(s.pos), s.box, s.periodic, 0)
    wantV = tbkpm.vac_moments(H, vx, a, b, r, M, 3, 0.1)
    cases = [(tbkpm.workspace_size(H, R, M, "c32"), tbkpm.least_workspace_size(H, R, M, "c32"), want,
              lambda: tbkpm.kpm_moments(H, a, b, r, M)),
             (tbkpm.workspace_size_batched(HB, R, M, "c32"), tbkpm.least_workspace_size_batched(HB, R, M, "c32"),
              wantB, lambda: tbkpm.kpm_moments_batched(HB, [a], [b], r, M)),
             (tbkpm.vac_workspace_size(H, R, M, "c32"), tbkpm.vac_workspace_size(H, R, M, "c32", least=True), wantV,
              lambda: tbkpm.vac_moments(H, vx, a, b, r, M, 3, 0.1))]
    for full, least, want, run in cases:
        assert full > least
        room(least + min(spare, (full - least) // 2))
        got = run()
        room(4 << 30)
        assert (got - want).abs().max().item() <= 1e-13 * max(s.n, want.abs().max().item())
