"""Assembly of rows on either side of the short-row rule, and the bounds of blocks
with several rows per thread or several structures.

Entries against the oracle: a hopping is one exp of a quotient of two rounded
distances, t_pair exp(-beta (r / r0 - 1)); the distances agree to a few eps and
beta r / r0 < 10, so values agree to about 40 eps, held to 1e-13.  Bounds from the
stored FP64 entries: sums of at most 12 terms in another order, 12 eps apart."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r_cut", [1.3, 2.0, 2.6, 2.95])     # 0 to 2, 3 to 4, 9 and 12 entries per row
@pytest.mark.parametrize("fmt,slice,sigma,reorder", [("sell_f64", 64, 0.06, True), ("csr_f64", 1, 0.12, False),
                                                     ("sell_f32", 256, 0.12, True), ("sell_f32", 1, 0.06, False)])
def test_short_and_long_rows(r_cut, fmt, slice, sigma, reorder):
    s = synth.graphene_sheet(13, 17, sigma, 4)
    H = G.build(s, fmt=fmt, slice=slice, reorder=reorder, r_cut=r_cut)
    csr, pairs = O.hamiltonian(s.pos, s.species, s.box, s.periodic, s.onsite, s.t_pair, r_cut=r_cut)
    orow, ocol, oval = G.csr_entries(csr)
    rows, cols, vals, _ = G.entries_in_atom_order(H)
    assert H.st.max_degree == np.diff(csr.row_ptr).max() and H.st.n_bonds == len(orow) // 2
    a, b = np.lexsort((cols, rows)), np.lexsort((ocol, orow))
    assert np.array_equal(np.asarray(rows)[a], orow[b]) and np.array_equal(np.asarray(cols)[a], ocol[b])
    tol = 1e-13 if fmt.endswith("f64") else 6.1e-8           # 1e-13 and half an ulp of FP32
    assert np.all(np.abs(np.asarray(vals)[a] - oval[b]) <= tol * np.abs(oval[b]))
    lo, hi = O.gershgorin(csr)
    assert H.bounds[0] == pytest.approx(lo, rel=1e-13) and H.bounds[1] == pytest.approx(hi, rel=1e-13)
    # stored order: ascending columns, padding (the row itself) after them
    t = H.tensors
    ptr, col, val = t["ptr"].cpu().numpy(), t["col"].cpu().numpy(), t["val"].cpu().numpy()
    C = H.st.slice if fmt != "csr_f64" else 1
    for q in range(0, len(ptr) - 1, 7):
        c = col[ptr[q]:ptr[q + 1]].reshape(-1, C)[:, :max(1, min(C, s.n - q * C))]
        v = val[ptr[q]:ptr[q + 1]].reshape(-1, C)[:, :c.shape[1]]
        for lane in range(c.shape[1]):
            real = v[:, lane] != 0
            k = int(real.sum())
            assert real[:k].all() and np.all(np.diff(c[:k, lane]) > 0)
            assert np.all(c[k:, lane] == q * C + lane)


def test_bounds_where_structures_meet_in_a_block():
    """Structures of a few atoms to several blocks: every structure's bounds are those of its own build."""
    ss = [synth.graphene_sheet(nx, ny, 0.05 + 0.01 * k, k) for k, (nx, ny) in
          enumerate([(2, 4), (3, 3), (9, 11), (2, 3), (40, 31), (5, 4)])]
    seg = np.concatenate([[0], np.cumsum([s.n for s in ss])])
    pos = np.concatenate([s.pos for s in ss])
    spc = np.concatenate([s.species for s in ss])
    H = tbkpm.build_hamiltonian_batched(G.to_dev(pos, torch.float64), G.to_dev(spc, torch.int32), seg,
                                        [s.box for s in ss], ss[0].periodic, ss[0].onsite, ss[0].t_pair, fmt="sell_f64")
    for k, s in enumerate(ss):
        one = G.build(s)
        assert tuple(H.bounds[k]) == tuple(one.bounds)


def test_bounds_of_several_rows_per_thread():
    """More than 4096 blocks of rows: the block's bounds cover all its rows."""
    s = synth.graphene_sheet(520, 521, 0.05, 2)
    assert s.n > 4096 * 256
    H = G.build(s, fmt="sell_f64", slice=64)
    ptr, val = H.tensors["ptr"], H.tensors["val"]
    n = s.n
    w = (ptr[1:] - ptr[:-1]) // 64
    asum = torch.zeros(len(w), 64, dtype=torch.float64, device=G.DEV)
    for k in range(int(w.max())):
        m = w > k
        at = ptr[:-1][m][:, None] + 64 * k + torch.arange(64, device=G.DEV)
        row = torch.nonzero(m)[:, 0][:, None] * 64 + torch.arange(64, device=G.DEV)
        asum[m] += torch.where(row < n, val[at].abs(), 0.0)
    hi = asum.reshape(-1)[:n].max().item()
    assert H.bounds[1] == pytest.approx(hi, rel=12 * 2.3e-16) and H.bounds[0] == pytest.approx(-hi, rel=12 * 2.3e-16)
