"""Performance cases of the library: what a density-of-states or transport run has it do.

Every case goes through the public binding (paper_2509_06525_amd.tbkpm) the way the benchmark and the
tests do.  Five kinds of work, picked by use:

  dos        one finite-temperature frame: Hamiltonian build, Chebyshev moments, DOS on 2001 energies
  moments    Chebyshev moments on a Hamiltonian that is already there (more vectors, more moments)
  snapshots  a stack of uneven snapshots: build (plain or learned hoppings), moments, DOS of each
  vac        velocity operator, correlation moments and running conductivity
  train      epochs of the hopping network on bond features

Sizes span the configurations of synth.WORKLOADS and the tests: from the 2,304-atom FP64 sheet (launches and
host time) to the 100 M-atom sheet (HBM), one vector to 32, odd vector counts and ragged sheets, FP64 and
complex-float vectors, CSR, SELL, 4x4 and 9x9 blocks and the displacement form.

`exact` repeats the physics in 64-bit torch from the same positions, without the library.
"""
import math

import numpy as np
import torch

from paper_2509_06525_amd import synth, tbkpm

DEV = "cuda"
CELL_X, CELL_Y = 4.26, math.sqrt(3.0) * 1.42
T_CC, BETA, R0, R_HOP = -2.7, 3.37, 1.42, 2.0
LZ = 20.0
HBAR = 0.6582119569
ONSITE = (0.0, 2.3, -1.9)
T_PAIR = ((-2.7, -2.2, -2.5), (-2.2, 0.0, -2.6), (-2.5, -2.6, 0.0))
SK_V, SK_ES, SK_EP = (-5.7, 5.4, 6.2, -2.7), -7.3, 0.0
SK_D, SK_ED = (-3.1, -2.4, 1.3, -1.9, 1.05, -0.21), 6.5
N_E = 2001


def listed():
    return [
        # the small FP64 check every installation starts with: launches, host round trips, allocations
        dict(name="dos_pristine_2304_f64", kind="dos", nx=24, ny=24, sigma=0.0, fmt="csr_f64", slice=1, R=4, M=256),
        # a ragged mid-size sheet with an odd number of vectors
        dict(name="moments_30k_r3", kind="moments", nx=83, ny=91, sigma=0.05, fmt="sell_f32", slice=256, R=3, M=512),
        # the 1 M-atom finite-temperature frame, 16 vectors at once
        dict(name="dos_thermal_1M_r16", kind="dos", nx=500, ny=500, sigma=0.05, fmt="sell_f32", slice=32, R=16,
             M=1000),
        # the 4 M-atom heterostructure: three species, onsite energies, 32 vectors
        dict(name="moments_stripes_4M_r32", kind="moments", nx=1000, ny=1000, sigma=0.03, stripes=True,
             fmt="sell_f32", slice=16, R=32, M=200),
        # the headline: 100 M atoms, one vector
        dict(name="dos_pristine_100M_r1", kind="dos", nx=5000, ny=5000, sigma=0.0, fmt="sell_f32", slice=256, R=1,
             M=500),
        # the FP64 path on an ordinary sheet, odd vector count
        dict(name="moments_250k_f64_r5", kind="moments", nx=250, ny=251, sigma=0.05, fmt="sell_f64", slice=64, R=5,
             M=300),
        # uneven snapshots (1k to 50k atoms) with the plain formula
        dict(name="snapshots_96_r8", kind="snapshots", count=96, n_min=1000, n_max=50000, learned=False, R=8, M=512),
        # the same kind of stack with the network's hoppings
        dict(name="snapshots_learned_48_r8", kind="snapshots", count=48, n_min=1000, n_max=50000, learned=True, R=8,
             M=256),
        # s, p orbitals: 4x4 blocks, 800,000 orbital rows
        dict(name="moments_sp3_200k_r16", kind="moments", nx=200, ny=250, sigma=0.05, orbitals=4, r_cut=2.0,
             fmt="bsell4_f32", slice=64, R=16, M=128),
        # s, p, d orbitals with third neighbours in the displacement form, 9,000,000 orbital rows
        dict(name="moments_spd_3nn_1M_r1", kind="moments", nx=500, ny=500, sigma=0.05, orbitals=9, r_cut=3.0,
             fmt="bgeom_f32", slice=256, R=1, M=64),
        # conductivity of a 250 k-atom sheet, 32 time steps of 0.1 fs
        dict(name="vac_250k", kind="vac", nx=250, ny=250, sigma=0.05, R=1, M=256, n_t=32, dt=0.1),
        # two epochs of the hopping network in minibatches of 2048 bonds
        dict(name="train_60k_bonds", kind="train", count=3, n_min=8000, n_max=20000, batch=2048, epochs=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sheet(rng, lo, hi):
    """Cells of a sheet with lo..hi atoms and an aspect ratio of 1/2 .. 2 (in length)."""
    n = _log(rng, lo, hi)
    ratio = rng.uniform(0.5, 2.0)
    nx = max(4, int(round(math.sqrt(n / 4.0 * ratio * CELL_Y / CELL_X))))
    return nx, max(6, int(round(n / 4.0 / nx)))


def draw(rng):
    kind = rng.choice(["dos", "dos", "moments", "moments", "moments", "orbitals", "snapshots", "vac", "train"])
    if kind == "train":
        return dict(kind="train", count=rng.randint(1, 4), n_min=1000, n_max=_log(rng, 4000, 20000),
                    batch=rng.choice([512, 1024, 2048, 3000]), epochs=rng.randint(1, 2))
    if kind == "vac":
        nx, ny = _sheet(rng, 2000, 400000)
        return dict(kind="vac", nx=nx, ny=ny, sigma=rng.uniform(0.02, 0.06), R=rng.choice([1, 1, 2, 3]),
                    M=_log(rng, 64, 256), n_t=rng.randint(8, 33), dt=0.1)
    if kind == "snapshots":
        return dict(kind="snapshots", count=_log(rng, 3, 96), n_min=1000, n_max=_log(rng, 5000, 50000),
                    learned=rng.random() < 0.4, R=rng.choice([1, 3, 4, 8, 8]), M=_log(rng, 64, 512))
    if kind == "orbitals":
        orb = rng.choice([4, 9])
        geom = rng.random() < 0.4
        nx, ny = _sheet(rng, 2000, 200000 if orb == 4 else 100000)
        return dict(kind="moments", nx=nx, ny=ny, sigma=rng.uniform(0.02, 0.06), orbitals=orb,
                    r_cut=3.0 if geom else 2.0, fmt="bgeom_f32" if geom else rng.choice(["bsell4_f32", "bsell4_f32",
                                                                                        "bsell4_f64"]),
                    slice=rng.choice([32, 64, 256]), R=rng.choice([1, 1, 2, 4, 8, 16]), M=_log(rng, 48, 200))
    fmt = rng.choice(["sell_f32", "sell_f32", "sell_f32", "sell_f64", "csr_f64"])
    nx, ny = _sheet(rng, 1000, 4000000 if fmt == "sell_f32" else 500000)
    n = 4 * nx * ny
    R = rng.choice([r for r in (1, 1, 2, 3, 4, 7, 8, 16, 32) if r * n <= 32000000])
    c = dict(kind=kind, nx=nx, ny=ny, sigma=rng.choice([0.0, rng.uniform(0.02, 0.08)]), fmt=fmt,
             slice=1 if fmt == "csr_f64" else rng.choice([16, 32, 64, 256]), R=R, M=_log(rng, 64, 1000))
    c["M"] = min(c["M"], max(64, int(4e9 / (n * R))))
    if kind == "moments":
        if rng.random() < 0.3:
            c["stripes"] = True
        if rng.random() < 0.25:
            c["doubling"] = True
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & (2**62 - 1))
    return g


def _positions(nx, ny, sigma, g):
    basis = torch.tensor([[0.0, 0.0], [0.71, 0.5 * CELL_Y], [2.13, 0.5 * CELL_Y], [2.84, 0.0]], dtype=torch.float64,
                         device=DEV)
    pos = torch.empty((ny, nx, 4, 3), dtype=torch.float64, device=DEV)
    pos[..., 0] = torch.arange(nx, dtype=torch.float64, device=DEV)[None, :, None] * CELL_X + basis[None, None, :, 0]
    pos[..., 1] = torch.arange(ny, dtype=torch.float64, device=DEV)[:, None, None] * CELL_Y + basis[None, None, :, 1]
    pos[..., 2] = 0.5 * LZ
    pos = pos.reshape(-1, 3)
    if sigma > 0.0:
        pos += sigma * torch.randn(pos.shape, dtype=torch.float64, device=DEV, generator=g)
    return pos


def _species(nx, ny, stripes):
    if not stripes:
        return torch.zeros(4 * nx * ny, dtype=torch.int32, device=DEV)
    cx = torch.arange(nx, device=DEV)[None, :, None].expand(ny, nx, 4)
    b = torch.arange(4, device=DEV)[None, None, :].expand(ny, nx, 4)
    sp = torch.where((cx // 50) % 2 == 1, 1 + b % 2, torch.zeros_like(b))
    return sp.reshape(-1).to(torch.int32).contiguous()


def _phases(n, R, dtype, g):
    phi = 2.0 * math.pi * torch.rand((n, R), dtype=torch.float64, device=DEV, generator=g)
    return torch.polar(torch.ones_like(phi), phi).to(dtype)


def _prec(fmt):
    return ("c32", torch.complex64) if fmt.endswith("f32") else ("f64", torch.complex128)


def _model(case):
    return (ONSITE, T_PAIR) if case.get("stripes") else ((0.0,), ((T_CC,),))


def _box(case):
    return (case["nx"] * CELL_X, case["ny"] * CELL_Y, LZ)


def _build(case, pos, sp, into=None):
    if case.get("orbitals"):
        kw = dict(r_cut=case["r_cut"], fmt=case["fmt"], slice=case["slice"])
        if case["orbitals"] == 9:
            kw.update(d=SK_D, e_d=SK_ED)
        return tbkpm.build_hamiltonian_sk(pos, sp, _box(case), (1, 1, 0), *SK_V, SK_ES, SK_EP, **kw)
    onsite, t_pair = _model(case)
    return tbkpm.build_hamiltonian(pos, sp, _box(case), (1, 1, 0), onsite, t_pair, fmt=case["fmt"],
                                   slice=case["slice"], into=into)


def _snapshot_sizes(case, seed):
    # sizes uniform in log, the same for every seed, so that every state of a case is the same amount of work
    sizes = np.exp(np.linspace(math.log(case["n_min"]), math.log(case["n_max"]), case["count"] + 2)[1:-1])
    sigmas = np.random.default_rng(int(seed) + 17).uniform(0.02, 0.08, size=case["count"])
    return [synth.sheet_dims_for(s) for s in sizes], sigmas


def _stack(case, seed, g):
    dims, sigmas = _snapshot_sizes(case, seed)
    parts = [_positions(nx, ny, float(s), g) for (nx, ny), s in zip(dims, sigmas)]
    seg = [0]
    for p in parts:
        seg.append(seg[-1] + p.shape[0])
    boxes = [(nx * CELL_X, ny * CELL_Y, LZ) for nx, ny in dims]
    return torch.cat(parts).contiguous(), seg, boxes


def _inputs(case, seed):
    """What `prepare` and `exact` share: positions, species, start vectors (or the stack)."""
    g = _gen(seed)
    if case["kind"] in ("snapshots", "train"):
        pos, seg, boxes = _stack(case, seed, g)
        r = _phases(pos.shape[0], case["R"], torch.complex64, g) if case["kind"] == "snapshots" else None
        return pos, seg, boxes, r
    pos = _positions(case["nx"], case["ny"], case["sigma"], g)
    sp = _species(case["nx"], case["ny"], case.get("stripes"))
    fmt = "sell_f32" if case["kind"] == "vac" else case["fmt"]
    r = _phases(pos.shape[0] * (case.get("orbitals") or 1), case["R"], _prec(fmt)[1], g)
    return pos, sp, r


def _energies(lo=-8.0, hi=8.0):
    return torch.linspace(lo, hi, N_E, dtype=torch.float64, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("snapshots", "train"):
        pos, seg, boxes, r = _inputs(case, seed)
        sp = torch.zeros(pos.shape[0], dtype=torch.int32, device=DEV)
        st = dict(case=case, pos=pos, sp=sp, seg=seg, boxes=boxes, r=r)
        if kind == "train" or case["learned"]:
            v = tbkpm.descriptor(pos, seg, boxes, (1, 1, 0))
            bonds = tbkpm.bonds(pos, seg, boxes, (1, 1, 0))
            st["shift"], st["scale"] = tbkpm.feature_moments(bonds, v)
            st["params"] = torch.from_numpy(synth.init_mlp_params(int(seed) % 1000 + 1)).to(DEV)
            if kind == "train":
                st["X"] = tbkpm.bond_features(bonds, v, st["shift"], st["scale"])
                st["y"] = tbkpm.coordination_target(bonds, v, synth.COORD_KAPPA, synth.COORD_Z0)
                return st
        if case["learned"]:
            H = tbkpm.build_hamiltonian_learned(pos, sp, seg, boxes, (1, 1, 0), [0.0], [[T_CC]], st["params"],
                                                st["shift"], st["scale"], slice=32)
        else:
            H = tbkpm.build_hamiltonian_batched(pos, sp, seg, boxes, (1, 1, 0), [0.0], [[T_CC]], slice=32)
        st["H"] = H
        st["work"] = torch.empty(tbkpm.workspace_size_batched(H, case["R"], case["M"], "c32"), dtype=torch.uint8,
                                 device=DEV)
        st["E"] = _energies().repeat(len(boxes), 1)
        return st
    pos, sp, r = _inputs(case, seed)
    c = dict(case, fmt="sell_f32", slice=256) if kind == "vac" else case
    H = _build(c, pos, sp)
    a, b = H.scale()
    st = dict(case=c, pos=pos, sp=sp, r=r, H=H, a=a, b=b, E=_energies())
    if kind != "vac":
        prec = _prec(c["fmt"])[0]
        cfg = None
        if case.get("doubling"):
            cfg = tbkpm.with_doubling(tbkpm.default_config(H, case["R"], prec))
        st["config"] = cfg
        st["work"] = tbkpm.alloc_workspace(H, case["R"], case["M"], prec, config=cfg)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "train":
        tr = tbkpm.MlpTrainer(st["params"].clone())
        hist = tr.train(st["X"], st["y"], case["epochs"], case["batch"], lr=2e-3, wd=1e-5, shuffle_seed=5)
        return dict(loss=hist, params=tr.params, m=tr.m, v=tr.v)
    if kind == "snapshots":
        if case["learned"]:
            H = tbkpm.build_hamiltonian_learned(st["pos"], st["sp"], st["seg"], st["boxes"], (1, 1, 0), [0.0],
                                                [[T_CC]], st["params"], st["shift"], st["scale"], slice=32,
                                                into=st["H"])
        else:
            H = tbkpm.build_hamiltonian_batched(st["pos"], st["sp"], st["seg"], st["boxes"], (1, 1, 0), [0.0],
                                                [[T_CC]], slice=32)
        st["H"] = H
        a, b = H.scales()
        mu = tbkpm.kpm_moments_batched(H, a, b, st["r"], case["M"], "c32", work=st["work"])
        return dict(mu=mu, rho=tbkpm.kpm_dos_batched(tbkpm.mean_moments(mu), a, b, st["E"]))
    if kind == "vac":
        H, a, b = st["H"], st["a"], st["b"]
        vx = tbkpm.build_velocity(H, st["pos"], _box(case), (1, 1, 0), 0)
        nu = tbkpm.vac_moments(H, vx, a, b, st["r"], case["M"], case["n_t"], case["dt"])
        mean = tbkpm.mean_moments(nu)
        return dict(nu=nu, sigma=tbkpm.vac_sigma(mean, a, b, case["dt"], st["E"]))
    prec = _prec(case["fmt"])[0]
    if kind == "dos":
        H = st["H"] = _build(case, st["pos"], st["sp"], into=st["H"])
        a, b = H.scale()
    else:
        H, a, b = st["H"], st["a"], st["b"]
    mu = tbkpm.kpm_moments(H, a, b, st["r"], case["M"], prec, work=st["work"], config=st["config"])
    if kind == "moments":
        return dict(mu=mu)
    return dict(mu=mu, rho=tbkpm.kpm_dos(tbkpm.mean_moments(mu), a, b, st["E"]))


# ---------------------------------------------------------------------------
# the least work
# ---------------------------------------------------------------------------

def work(case):
    """Inputs read once, outputs written once; the recurrence's multiply-adds."""
    kind, M = case["kind"], case.get("M", 0)
    if kind in ("snapshots", "train"):
        dims, _ = _snapshot_sizes(case, 0)
        n = sum(4 * nx * ny for nx, ny in dims)
    else:
        n = 4 * case["nx"] * case["ny"]
    if kind == "train":
        nb = 1.5 * n
        return dict(bytes=case["epochs"] * nb * 36 + 6 * 4 * 1633, flops=case["epochs"] * nb * 3 * 2 * 1600)
    R = case["R"]
    orb = case.get("orbitals") or 1
    deg = 12 if case.get("r_cut", 2.0) > 2.5 else 3
    per_row = 2 * 2 * deg * orb + 4 + 4                      # H x, the recurrence, the overlap
    if kind == "snapshots":
        return dict(bytes=n * (28 + 8 * R) + 8 * len(dims) * (R * M + 2 * N_E),
                    flops=n * R * M * per_row + len(dims) * N_E * M * 3 + (n * 1.5 * 3200 if case["learned"] else 0))
    if kind == "vac":
        a, n_t = 8.5 * 1.4, case["n_t"]
        terms = a * case["dt"] / HBAR + 14
        return dict(bytes=n * (8 * deg + 24 + 8 * R) + 8 * n_t * (R * M + N_E),
                    flops=n * R * n_t * (M * per_row + 2 * terms * (4 * deg + 12)) + n_t * N_E * M * 3)
    cplx = 8 if _prec(case["fmt"])[0] == "c32" else 16
    mu = 8 * R * M
    if kind == "dos":
        return dict(bytes=n * (28 + cplx * R) + mu + 16 * N_E, flops=n * R * M * per_row + N_E * M * 3)
    half = cplx // 2
    if case["fmt"].startswith("bgeom"):
        h = n * deg * 16
    elif orb > 1:
        h = n * deg * (4 + orb * orb * half)
    else:
        h = n * deg * (4 + half)
    return dict(bytes=h + n * orb * (4 + cplx * R) + mu, flops=n * orb * R * M * per_row)


# ---------------------------------------------------------------------------
# 64-bit values
# ---------------------------------------------------------------------------

def _neighbours(pos, nx, ny, r_cut):
    """(idx [n][W], displacement [n][W][3], r [n][W], mask [n][W]) within r_cut, from the 3 x 3 cells around."""
    n = pos.shape[0]
    box = torch.tensor([nx * CELL_X, ny * CELL_Y], dtype=torch.float64, device=DEV)
    at = torch.arange(n, device=DEV)
    cx, cy = (at // 4) % nx, at // (4 * nx)
    found, count = [], torch.zeros(n, dtype=torch.long, device=DEV)
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            cell = ((cy + dy) % ny) * nx + (cx + dx) % nx
            for b in range(4):
                j = 4 * cell + b
                d = pos[j] - pos
                d[:, :2] -= box * torch.round(d[:, :2] / box)
                r = d.norm(dim=1)
                ok = (r < r_cut) & (j != at)
                found.append((at[ok], j[ok], d[ok], r[ok], count[ok]))
                count += ok
    W = int(count.max())
    idx = at[:, None].repeat(1, W)
    disp = torch.zeros((n, W, 3), dtype=torch.float64, device=DEV)
    rr = torch.full((n, W), R0, dtype=torch.float64, device=DEV)
    mask = torch.zeros((n, W), dtype=torch.bool, device=DEV)
    for i, j, d, r, k in found:
        idx[i, k], disp[i, k], rr[i, k], mask[i, k] = j, d, r, True
    return idx, disp, rr, mask


class _Exact:
    """H as its rows' neighbour values; `apply` is H x for x [n][R] complex128."""

    def __init__(self, case, pos, sp):
        self.orb = case.get("orbitals") or 1
        nx, ny = case["nx"], case["ny"]
        if case["sigma"] == 0.0 and not case.get("stripes") and self.orb == 1:
            self.lattice, self.shape = True, (ny, nx, 4)
            self.bounds = (3 * T_CC, -3 * T_CC)
            return
        self.lattice = False
        self.idx, self.disp, r, mask = _neighbours(pos, nx, ny, case.get("r_cut", R_HOP))
        f = torch.exp(-BETA * (r / R0 - 1.0)) * mask
        if self.orb == 1:
            onsite, t_pair = _model(case)
            t = torch.tensor(t_pair, dtype=torch.float64, device=DEV)
            s = sp.long()
            self.val = t[s[:, None], s[self.idx]] * f
            self.on = torch.tensor(onsite, dtype=torch.float64, device=DEV)[s]
            off = self.val.abs().sum(1)
        else:
            c = self.disp / torch.where(mask, r, torch.ones_like(r))[..., None]
            self.val = [(_sk_block(c[:, k], self.orb) * f[:, k, None, None]).contiguous() for k in range(r.shape[1])]
            e = [SK_ES] + [SK_EP] * 3 + [SK_ED] * 5
            self.on = torch.tensor(e[:self.orb], dtype=torch.float64, device=DEV).repeat(pos.shape[0])
            off = sum(v.abs().sum(2) for v in self.val).reshape(-1)
        self.bounds = (float((self.on - off).min()), float((self.on + off).max()))

    def scale(self):
        lo, hi = self.bounds
        return 1.01 * (hi - lo) / 2.0, (hi + lo) / 2.0

    def apply(self, x):
        if self.lattice:
            v = x.reshape(*self.shape, -1)
            x0, x1, x2, x3 = v.unbind(2)
            y = torch.empty_like(v)
            y[:, :, 0] = x1 + torch.roll(x1, 1, 0) + torch.roll(x3, 1, 1)
            y[:, :, 1] = x0 + torch.roll(x0, -1, 0) + x2
            y[:, :, 2] = x3 + torch.roll(x3, -1, 0) + x1
            y[:, :, 3] = x2 + torch.roll(x2, 1, 0) + torch.roll(x0, -1, 1)
            return y.mul_(T_CC).reshape(x.shape)
        if self.orb == 1:
            y = self.on[:, None] * x
            for k in range(self.idx.shape[1]):
                y.addcmul_(self.val[:, k, None].to(x.dtype), x[self.idx[:, k]])
            return y
        n, R = self.idx.shape[0], x.shape[1]
        xr = torch.view_as_real(x).reshape(n, self.orb, 2 * R)
        y = (self.on[:, None] * x)
        acc = torch.view_as_real(y).reshape(n, self.orb, 2 * R)
        for k in range(self.idx.shape[1]):
            acc += torch.bmm(self.val[k], xr[self.idx[:, k]].contiguous())
        return torch.view_as_complex(acc.reshape(n * self.orb, R, 2).contiguous())

    def moments(self, r, left, a, b, M):
        """Re <left|T_m r> per vector: [R][M]."""
        mu = torch.empty((r.shape[1], M), dtype=torch.float64, device=DEV)

        def dot(t):
            return (torch.view_as_real(left) * torch.view_as_real(t)).sum(dim=(0, 2))

        def ht(x):
            y = self.apply(x)
            return y.div_(a) if b == 0.0 else y.sub_(x, alpha=b).div_(a)

        t0, t1 = r, ht(r)
        mu[:, 0] = dot(t0)
        mu[:, 1] = dot(t1)
        for m in range(2, M):
            t0, t1 = t1, ht(t1).mul_(2.0).sub_(t0)
            mu[:, m] = dot(t1)
        return mu


def _sk_block(c, orb):
    """Slater-Koster blocks [n][orb][orb] for direction cosines c [n][3] (projector form)."""
    n = c.shape[0]
    ss, sp, pps, ppp = SK_V
    B = torch.zeros((n, orb, orb), dtype=torch.float64, device=DEV)
    eye3 = torch.eye(3, dtype=torch.float64, device=DEV)
    cc = c[:, :, None] * c[:, None, :]
    B[:, 0, 0] = ss
    B[:, 0, 1:4] = sp * c
    B[:, 1:4, 0] = -sp * c
    B[:, 1:4, 1:4] = pps * cc + ppp * (eye3 - cc)
    if orb == 4:
        return B
    sd, pds, pdp, dds, ddp, ddd = SK_D
    s3 = math.sqrt(3.0)
    l, m, k = c.unbind(1)
    o = torch.zeros_like(l)
    # u: the d orbitals' sigma amplitudes along c; J = du/dc
    u = torch.stack([s3 * l * m, s3 * m * k, s3 * k * l, 0.5 * s3 * (l * l - m * m), k * k - 0.5 * (l * l + m * m)], 1)
    J = torch.stack([torch.stack([s3 * m, s3 * l, o], 1), torch.stack([o, s3 * k, s3 * m], 1),
                     torch.stack([s3 * k, o, s3 * l], 1), torch.stack([s3 * l, -s3 * m, o], 1),
                     torch.stack([-l, -m, 2.0 * k], 1)], 1)
    cu = c[:, :, None] * u[:, None, :]
    pd = pds * cu + pdp * (J.transpose(1, 2) - 2.0 * cu) / s3
    uu = u[:, :, None] * u[:, None, :]
    Jc = (J * c[:, None, :]).sum(2)
    JJ = sum(J[:, :, q, None] * J[:, None, :, q] for q in range(3)) - Jc[:, :, None] * Jc[:, None, :]
    eye5 = torch.eye(5, dtype=torch.float64, device=DEV)
    B[:, 0, 4:] = sd * u
    B[:, 4:, 0] = sd * u
    B[:, 1:4, 4:] = pd
    B[:, 4:, 1:4] = -pd.transpose(1, 2)
    B[:, 4:, 4:] = ddd * eye5 + (dds - ddd) * uu + (ddp - ddd) * JJ / 3.0
    return B


def _jackson(M):
    n = torch.arange(M, dtype=torch.float64, device=DEV)
    q = math.pi / (M + 1)
    return ((M - n + 1) * torch.cos(q * n) + torch.sin(q * n) / math.tan(q)) / (M + 1)


def _dos(mu, a, b, E):
    """Jackson-damped density of states [..][nE] from moments [..][M]."""
    M = mu.shape[-1]
    x = (E - b) / a
    ok = x.abs() < 1.0
    th = torch.arccos(torch.where(ok, x, torch.zeros_like(x)))
    w = _jackson(M) * mu
    w = torch.cat([w[..., :1], 2.0 * w[..., 1:]], -1)
    T = torch.cos(torch.arange(M, dtype=torch.float64, device=DEV)[:, None] * th[None, :])
    return torch.where(ok, (w @ T) / (a * math.pi * torch.sqrt(1.0 - x * x)), torch.zeros_like(x))


def _bessel(k, z):
    """J_k(z) from its integral (the trapezoidal rule is exact to rounding on a period)."""
    th = np.linspace(0.0, 2.0 * np.pi, 4096, endpoint=False)
    return float(np.mean(np.cos(k * th - z * np.sin(th))))


def _vac(case, H, pos, r, a, b):
    hb = HBAR
    velocity = (H.val * H.disp[..., 0] / hb) if not H.lattice else None
    n_t, M, R = case["n_t"], case["M"], r.shape[1]

    def V(x):
        y = torch.zeros_like(x)
        for k in range(H.idx.shape[1]):
            y.addcmul_(velocity[:, k, None].to(x.dtype), x[H.idx[:, k]])
        return 1j * y

    z = a * case["dt"] / hb
    coef = []
    for k in range(10000):
        j = _bessel(k, z)
        coef.append((1.0 if k == 0 else 2.0) * j * (-1j) ** k)
        if k > z and abs(j) < 1e-16:
            break
    phase = complex(math.cos(b * case["dt"] / hb), -math.sin(b * case["dt"] / hb))

    def evolve(x):
        t0, t1 = x, (H.apply(x) - b * x) / a
        acc = coef[0] * t0 + coef[1] * t1
        for ck in coef[2:]:
            t0, t1 = t1, 2.0 * (H.apply(t1) - b * t1) / a - t0
            acc += ck * t1
        return phase * acc

    phi = torch.cat([r, V(r)], 1)
    start, left = [], []
    for j in range(n_t):
        start.append(V(phi[:, :R].contiguous()))
        left.append(phi[:, R:].clone())
        if j + 1 < n_t:
            phi = evolve(phi)
    nu = torch.cat([H.moments(torch.cat(start[q:q + 8], 1), torch.cat(left[q:q + 8], 1), a, b, M)
                    for q in range(0, n_t, 8)])
    nu = nu.reshape(n_t, R, M)
    C = _dos(nu.mean(1), a, b, _energies())
    sigma = torch.zeros_like(C)
    sigma[1:] = torch.cumsum(0.5 * case["dt"] * (C[1:] + C[:-1]), 0)
    return dict(nu=nu, sigma=sigma)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train" or case.get("learned"):
        return None                      # bfloat16 products: no 64-bit value
    if kind == "snapshots":
        pos, seg, boxes, r = _inputs(case, seed)
        dims, sigmas = _snapshot_sizes(case, seed)
        mu, rho = [], []
        for s, (nx, ny) in enumerate(dims):
            part = slice(seg[s], seg[s + 1])
            H = _Exact(dict(nx=nx, ny=ny, sigma=float(sigmas[s])), pos[part],
                       torch.zeros(seg[s + 1] - seg[s], dtype=torch.int32, device=DEV))
            a, b = H.scale()
            x = r[part].to(torch.complex128)
            mu.append(H.moments(x, x, a, b, case["M"]))
            rho.append(_dos(mu[-1].mean(0), a, b, _energies()))
        return dict(mu=torch.stack(mu), rho=torch.stack(rho))
    pos, sp, r = _inputs(case, seed)
    H = _Exact(case, pos, sp)
    a, b = H.scale()
    x = r.to(torch.complex128)
    if kind == "vac":
        return _vac(case, H, pos, x, a, b)
    mu = H.moments(x, x, a, b, case["M"])
    if kind == "moments":
        return dict(mu=mu)
    return dict(mu=mu, rho=_dos(mu.mean(0), a, b, _energies()))
