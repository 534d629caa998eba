"""Performance cases of the polarization path: what programs that use this
framework have it do, at the sizes of its workloads.

Every case is a synthetic water system like those of the benchmark and the
tests: five sites per water (O, H1, H2 and the two O-H barycentres) with
random dipoles, quadrupoles and polarizabilities, at 1 g/cm^3 on a jittered
lattice (periodic) or as a compact piece of it (cluster).  The kinds are

  evaluate  new positions, a cold solve, energies and all forces (optionally
            with molecular local frames and the virial);
  step      new positions, a solve warm-started from the previous step's
            dipoles, energies and all forces (a step of dynamics, or a
            repeated request of a server);
  field     new positions, the permanent field;
  matvec    T p on a resident system, for a caller's own solver;
  tcg       new positions, truncated conjugate gradient, E_pol;
  batch     many gas-phase clusters in one call.

`exact` evaluates the same quantities in FP64 with plain torch: pair sums
over an explicit pair list, SPME with torch's FFT, a conjugate gradient far
below the tolerance, and forces by automatic differentiation.
"""
import math

import numpy as np
import torch

from paper_2201_00804_amd import Engine, default_params

DEBYE = 4.803204
COULOMB = 332.0637133
THOLE = 0.28
TOL = 1e-8            # D, the tolerance of the benchmark
VOLUME = 29.95        # A^3 per water
DEV = "cuda"


def listed():
    return [
        # one water dimer: the smallest call, all latency
        dict(name="batch1_dimer_fp64", kind="batch", clusters=1, lo=2, hi=2, precision="fp64"),
        # what the server's cluster worker sends: 2 to 64 waters each
        dict(name="batch48_mixed", kind="batch", clusters=48, lo=2, hi=64, precision="mixed"),
        # a data set of small clusters evaluated at once
        dict(name="batch700_fp64", kind="batch", clusters=700, lo=2, hi=8, precision="fp64"),
        # one gas-phase cluster through a context of its own
        dict(name="cluster80_fp64", kind="evaluate", nx=0, ny=0, nz=0, waters=80,
             precision="fp64", precond="molblock", frames=False),
        # the dynamics box of the paper, one warm-started step
        dict(name="box216_step_fp64", kind="step", nx=6, ny=6, nz=6, waters=216,
             precision="fp64", precond="molblock"),
        # a box with unequal sides, local frames and the virial (constant
        # pressure), the default preconditioner
        dict(name="box1001_frames_fp64", kind="evaluate", nx=7, ny=11, nz=13, waters=1001,
             precision="fp64", precond="diag", frames=True),
        # the fixed-cost solver
        dict(name="box1024_tcg_fp64", kind="tcg", nx=8, ny=8, nz=16, waters=1024,
             precision="fp64", precond="diag"),
        # the server's largest box
        dict(name="box4096_mixed", kind="evaluate", nx=16, ny=16, nz=16, waters=4096,
             precision="mixed", precond="molblock", frames=False),
        # the benchmark workload in both precisions
        dict(name="box32000_mixed", kind="evaluate", nx=32, ny=32, nz=32, waters=32000,
             precision="mixed", precond="molblock", frames=False),
        dict(name="box32000_fp64", kind="evaluate", nx=32, ny=32, nz=32, waters=32000,
             precision="fp64", precond="molblock", frames=False),
        # the largest box
        dict(name="box96000_field_mixed", kind="field", nx=46, ny=46, nz=46, waters=96000,
             precision="mixed", precond="diag"),
        # one operator application for a caller's own solver
        dict(name="box32000_matvec_fp64", kind="matvec", nx=32, ny=32, nz=32, waters=32000,
             precision="fp64", precond="diag"),
    ]


def draw(rng):
    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    precision = rng.choice(["fp64", "mixed"])
    kind = rng.choice(["batch", "cluster", "evaluate", "evaluate", "step", "field", "matvec",
                       "tcg"])
    if kind == "batch":
        hi = log_uniform(2, 64)
        lo = rng.randint(1, hi)
        most = max(1, min(1000, 48 * 33 * 33 // (hi * hi)))
        return dict(kind="batch", clusters=log_uniform(1, most), lo=lo, hi=hi,
                    precision=precision)
    if kind == "cluster":
        return dict(kind="evaluate", nx=0, ny=0, nz=0, waters=log_uniform(8, 128),
                    precision=precision, precond=rng.choice(["diag", "molblock"]),
                    frames=rng.random() < 0.5)
    # box edges from 6 waters up, unequal ones among them
    n = log_uniform(216, 30000)
    side = n ** (1.0 / 3.0)
    nx = max(6, int(round(side * rng.uniform(0.8, 1.2))))
    ny = max(6, int(round(side * rng.uniform(0.8, 1.2))))
    nz = max(6, min(int(round(n / (nx * ny))), 30000 // (nx * ny)))
    waters = nx * ny * nz - rng.randint(0, nx * ny * nz // 50)
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, waters=waters, precision=precision,
             precond=rng.choice(["diag", "molblock"]))
    if kind == "evaluate":
        c["frames"] = rng.random() < 0.25
    return c


# ------------------------------------------------------------------ inputs
def _rotations(rng, n):
    """n uniformly random rotation matrices (normalised quaternions)."""
    w, x, y, z = rng.standard_normal((4, n))
    s = 2.0 / (w * w + x * x + y * y + z * z)
    return np.stack([1 - s * (y * y + z * z), s * (x * y - z * w), s * (x * z + y * w),
                     s * (x * y + z * w), 1 - s * (x * x + z * z), s * (y * z - x * w),
                     s * (x * z - y * w), s * (y * z + x * w), 1 - s * (x * x + y * y)],
                    axis=-1).reshape(n, 3, 3)


def _sites(rng, centres):
    """Waters at the centres with random orientations: [5 n, 3]."""
    h = math.radians(0.5 * 104.52)
    h1 = 0.9572 * np.array([math.sin(h), 0.0, math.cos(h)])
    h2 = h1 * np.array([-1.0, 1.0, 1.0])
    frame = np.stack([np.zeros(3), h1, h2, 0.5 * h1, 0.5 * h2])
    rot = _rotations(rng, len(centres))
    return (centres[:, None, :] + np.matmul(frame[None], rot.transpose(0, 2, 1))).reshape(-1, 3)


def _properties(rng, n_waters):
    n = 5 * n_waters
    v = rng.standard_normal((n, 3))
    dip = v / np.linalg.norm(v, axis=1, keepdims=True) * (0.1 * rng.random((n, 1)) ** (1 / 3))
    quad = rng.uniform(-0.1, 0.1, (n, 6))
    quad[:, 5] = -(quad[:, 0] + quad[:, 3])
    rot = _rotations(rng, n)
    a = np.matmul(rot * rng.uniform(0.3, 1.0, (n, 1, 3)), rot.transpose(0, 2, 1))
    alpha = a[:, [0, 0, 0, 1, 1, 2], [0, 1, 2, 1, 2, 2]]
    polarizable = np.tile([True, False, False, True, True], n_waters)
    alpha[~polarizable] = 0.0
    return dict(q=np.tile([-0.8, 0.4, 0.4, 0.0, 0.0], n_waters), dip=dip, quad=quad, alpha=alpha,
                mol=np.repeat(np.arange(n_waters, dtype=np.int32), 5))


def _cluster_sites(rng, n_waters):
    """The lattice points nearest to a random point, jittered."""
    m = int(math.ceil(n_waters ** (1 / 3))) + 2
    grid = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    centre = 0.5 * (m - 1) + rng.uniform(-0.5, 0.5, 3)
    near = np.argsort(((grid - centre) ** 2).sum(1), kind="stable")[:n_waters]
    c = (grid[np.sort(near)] - centre) * VOLUME ** (1 / 3)
    return _sites(rng, c + rng.uniform(-0.1, 0.1, c.shape))


def _system(case, seed):
    rng = np.random.default_rng(seed)
    if case["kind"] == "batch":   # the sizes are the case's, the rest the seed's
        sizes = np.random.default_rng([case["clusters"], case["lo"], case["hi"]]).integers(
            case["lo"], case["hi"] + 1, case["clusters"])
        pos = np.concatenate([_cluster_sites(rng, int(k)) for k in sizes])
        s = _properties(rng, int(sizes.sum()))
        s.update(pos=pos, box=None, sizes=sizes)
        s["mol"] = np.concatenate([np.repeat(np.arange(k, dtype=np.int32), 5) for k in sizes])
    elif case["nx"] == 0:
        s = _properties(rng, case["waters"])
        s.update(pos=_cluster_sites(rng, case["waters"]), box=None)
    else:
        dims = np.array([case["nx"], case["ny"], case["nz"]])
        total = int(dims.prod())
        spacing = (VOLUME * case["waters"] / total) ** (1 / 3)
        chosen = np.sort(rng.choice(total, case["waters"], replace=False))
        cell = np.stack([chosen % dims[0], chosen // dims[0] % dims[1],
                         chosen // (dims[0] * dims[1])], axis=1)
        c = (cell + 0.5) * spacing
        box = dims * spacing
        s = _properties(rng, case["waters"])
        s.update(pos=np.mod(_sites(rng, c + rng.uniform(-0.1, 0.1, c.shape)), box), box=box)
    if case.get("frames"):
        first = np.arange(len(s["pos"])) // 5 * 5
        s["frames"] = np.stack([first, first + 1, first + 2], 1).astype(np.int32)
    if case["kind"] == "step":   # the positions one step earlier
        s["pos0"] = s["pos"] + rng.uniform(-0.01, 0.01, s["pos"].shape)
    if case["kind"] == "matvec":
        s["p"] = 0.1 * rng.standard_normal(s["pos"].shape)
    return s


def _method(case, s):
    """Cutoff, Ewald parameter and grid of a box, as the named workloads
    have them (about 1 A per grid point)."""
    if s["box"] is None:
        return dict()
    small = s["box"].min() < 19.0

    def size(length):
        k = 2
        while True:
            m = k
            for f in (2, 3, 5):
                while m % f == 0:
                    m //= f
            if m == 1 and k >= 0.966 * length:
                return k
            k += 2

    return dict(cutoff=8.0 if small else 9.0, beta=0.45 if small else 0.40,
                grid=tuple(size(x) for x in s["box"]), order=5)


def _params(case, s):
    return default_params(tol=TOL, precision=case["precision"], thole_a=THOLE,
                          precond=case.get("precond", "diag"), **_method(case, s))


def _t(a, dtype=torch.float64):
    return torch.as_tensor(a, dtype=dtype, device=DEV).contiguous()


def prepare(case, seed):
    s = _system(case, seed)
    prm = _params(case, s)
    st = dict(case=case, pos=_t(s["pos"]))
    if case["kind"] == "batch":
        from paper_2201_00804_amd.batch import ClusterBatch
        st.update(batch=ClusterBatch(0), params=prm, mol=_t(s["mol"], torch.int32),
                  offsets=[0] + [int(x) for x in 5 * np.cumsum(s["sizes"])],
                  **{k: _t(s[k]) for k in ("q", "dip", "quad", "alpha")})
        return st
    eng = Engine(0)
    eng.set_system(_t(s.get("pos0", s["pos"])), _t(s["mol"], torch.int32), s["box"], prm)
    eng.set_multipoles(_t(s["q"]), _t(s["dip"]), _t(s["quad"]))
    eng.set_polarizabilities(_t(s["alpha"]))
    if case.get("frames"):
        eng.set_local_frames(_t(s["frames"], torch.int32), _t(s["dip"]), _t(s["quad"]),
                             _t(s["alpha"]))
    st["engine"] = eng
    if case["kind"] == "step":
        st["mu0"] = eng.solve()[0]
    if case["kind"] == "matvec":
        st["p"] = _t(s["p"])
        eng.permanent_field()   # sorted records and lists in place
    return st


def run(st):
    kind = st["case"]["kind"]
    if kind == "batch":
        r = st["batch"].run(st["offsets"], st["pos"], st["mol"], st["q"], st["dip"], st["quad"],
                            st["alpha"], st["params"])
        return dict(mu=r.mu, forces=r.forces, e_pol=r.e_pol, e_elec=r.e_elec)
    eng = st["engine"]
    if kind == "matvec":
        return dict(tp=eng.apply_T(st["p"]))
    if kind == "step":
        eng.set_dipoles(st["mu0"])
        eng.update_positions(st["pos"])
        mu, _, _ = eng.solve(warm_start=True)
        e_pol, e_elec, f = eng.energy_forces()
        return dict(e_pol=e_pol, e_elec=e_elec, forces=f, mu=mu)
    eng.update_positions(st["pos"])
    if kind == "field":
        return dict(field=eng.permanent_field())
    if kind == "tcg":
        mu, e_pol = eng.solve_tcg(2, omega=1.0)
        return dict(e_pol=e_pol, mu=mu)
    mu, _, _ = eng.solve()
    if st["case"]["frames"]:
        e_pol, e_elec, f, w = eng.energy_forces(virial=True)
        return dict(e_pol=e_pol, e_elec=e_elec, forces=f, mu=mu,
                    virial=torch.tensor(w, dtype=torch.float64))
    e_pol, e_elec, f = eng.energy_forces()
    return dict(e_pol=e_pol, e_elec=e_elec, forces=f, mu=mu)


def work(case):
    """Per site 23 doubles in and up to 6 out; per unordered pair within the
    cutoff 190 flops for the field and energy, 560 for the forces; per
    unordered polarizable pair 70 for its coefficients and 26 per operator
    application; SPME: 125 grid points per site and pass, 5 N log2 N per
    transform.  Counts of operator applications: those the solver is known
    to take on these systems."""
    kind = case["kind"]
    if kind == "batch":
        waters, per = case["clusters"] * 0.5 * (case["lo"] + case["hi"]), None
        sq = case["clusters"] * (case["lo"] ** 2 + case["lo"] * case["hi"] + case["hi"] ** 2) / 3.0
        pairs, pol = 12.5 * sq, 4.5 * sq
        grid = 0
    else:
        waters = case["waters"]
        per = 4.0 / 3.0 * math.pi * (9.0 if waters > 300 else 8.0) ** 3 / VOLUME
        per = min(per, waters) if case["nx"] else waters
        pairs, pol = 0.5 * 25.0 * waters * per, 0.5 * 9.0 * waters * per
        grid = VOLUME * waters if case["nx"] else 0
    n = 5 * waters
    fft = 10.0 * grid * math.log2(grid) if grid else 0.0
    recip = (lambda sites, terms: 250.0 * sites * terms + fft) if grid else (lambda *a: 0.0)
    field = 190.0 * pairs + recip(n, 10) + recip(0.6 * n, 3)
    matvec = 26.0 * pol + recip(0.6 * n, 6)
    forces = 560.0 * pairs + recip(n, 30)
    inputs, vec = n * 23 * 8.0, n * 3 * 8.0
    if kind == "field":
        return dict(bytes=inputs + vec, flops=field)
    if kind == "matvec":
        return dict(bytes=2 * vec + 0.6 * n * 9 * 8.0, flops=96.0 * pol + recip(0.6 * n, 6))
    if kind == "tcg":
        return dict(bytes=inputs + vec, flops=field + 70.0 * pol + 3 * matvec)
    iters = (14 if case.get("precond", "diag") == "diag" else 9) - (2 if kind == "step" else 0)
    return dict(bytes=inputs + 2 * vec, flops=field + forces + 70.0 * pol + (iters + 2) * matvec)


# ------------------------------------------------------------------ exact
def _pairs(x, box, rc, seg):
    """Unordered pairs (i, j): all of one segment (clusters), or closer than
    rc in the minimum image (periodic)."""
    n = len(x)
    if box is None:
        out = []
        off = torch.cat([torch.zeros(1, dtype=torch.long, device=x.device),
                         torch.bincount(seg).cumsum(0)]).tolist()
        for a, b in zip(off[:-1], off[1:]):
            out.append(torch.triu_indices(b - a, b - a, 1, device=x.device) + a)
        return torch.cat(out, 1)
    z, order = torch.sort(x[:, 2])
    length = float(box[2])
    out = []
    step = 2048
    for a in range(0, n, step):
        b = min(n, a + step)
        if float(z[b - 1] - z[a]) + 2 * rc >= length:
            cand = torch.arange(n, device=x.device)
        else:
            lo, hi = float(z[a]) - rc, float(z[b - 1]) + rc
            keep = (z >= lo) & (z <= hi) | (z >= lo + length) | (z <= hi - length)
            cand = torch.nonzero(keep).reshape(-1)
        r2 = 0.0
        for k in range(3):
            d = x[order[a:b], k, None] - x[order[cand], k][None]
            r2 = r2 + (d - box[k] * torch.round(d / box[k])) ** 2
        i, j = torch.nonzero(r2 < rc * rc, as_tuple=True)
        i, j = order[a + i], order[cand[j]]
        out.append(torch.stack([i, j])[:, i < j])
    return torch.cat(out, 1)


def _separation(x, i, j, box):
    r = x[i] - x[j]
    if box is not None:
        r = r - box * torch.round(r.detach() / box)
    return r


def _base(r, beta, top):
    """Ewald B_0..B_top, or the bare kernel for clusters (beta None)."""
    r2 = r * r
    if beta is None:
        c = [1 / r]
        for k in range(1, top + 1):
            c.append((2 * k - 1) * c[-1] / r2)
        return c
    g = torch.exp(-(beta * r) ** 2) / (beta * math.sqrt(math.pi))
    c = [torch.erfc(beta * r) / r]
    for k in range(1, top + 1):
        c.append(((2 * k - 1) * c[-1] + (2 * beta * beta) ** k * g) / r2)
    return c


def _thole(r, si, sj):
    """1 - lambda_(2n+1), n = 0..4 (0 for n = 0 and for unpolarizable sites)."""
    x = THOLE * r ** 3 * si * sj
    e = torch.exp(-x) * ((si > 0) & (sj > 0))
    return [torch.zeros_like(r), e, (1 + x) * e, (1 + x + 0.6 * x * x) * e,
            (1 + x + 18 / 35 * x * x + 9 / 35 * x ** 3) * e]


def _interaction(c, a, b, r):
    """Energy of multipoles a at r_i and b at r_j, r = r_i - r_j."""
    qa, da, ta = a
    qb, db, tb = b
    dot = lambda u, v: (u * v).sum(-1)   # noqa: E731
    ra, rb = (ta * r[:, None, :]).sum(-1), (tb * r[:, None, :]).sum(-1)
    dra, drb, rra, rrb = dot(da, r), dot(db, r), dot(ra, r), dot(rb, r)
    u = c[0] * qa * qb + c[1] * (qa * drb - qb * dra + dot(da, db))
    u = u + c[2] * ((qa * rrb + qb * rra) / 3 - dra * drb + 2 / 3 * (dot(da, rb) - dot(db, ra))
                    + 2 / 9 * (ta * tb).sum((-1, -2)))
    u = u + c[3] * ((drb * rra - dra * rrb) / 3 - 4 / 9 * dot(ra, rb))
    return u + c[4] * rra * rrb / 9


def _splines(x, box, grid, p):
    """Grid indices [n, 3, p] and B-spline values with two derivatives (with
    respect to the position), differentiable in x."""
    k = torch.tensor(grid, dtype=torch.float64, device=x.device)
    u = x * (k / box)
    base = torch.floor(u.detach())
    w = u - base
    idx = (base[:, :, None].long() - torch.arange(p, device=x.device)) % k[None, :, None].long()
    zero = torch.zeros_like(w)
    level = {1: [torch.ones_like(w)] + [zero] * (p - 1)}
    for m in range(2, p + 1):
        old = level[m - 1]
        level[m] = [((w + t) * old[t] + ((m - w - t) * old[t - 1] if t else zero)) / (m - 1)
                    for t in range(p)]
    at = lambda m, t: level[m][t] if t >= 0 else zero   # noqa: E731
    d0 = torch.stack(level[p], -1)
    d1 = torch.stack([at(p - 1, t) - at(p - 1, t - 1) for t in range(p)], -1)
    d2 = torch.stack([at(p - 2, t) - 2 * at(p - 2, t - 1) + at(p - 2, t - 2) for t in range(p)],
                     -1)
    s = (k / box)[None, :, None]
    return idx, (d0, d1 * s, d2 * s * s)


def _influence(box, grid, p, beta, dev):
    """The SPME influence function on the full grid."""
    lev = [0.0] * (p + 1)
    lev[1] = 1.0   # M_2 at the integers
    for m in range(3, p + 1):
        lev = [(t * lev[t] + (m - t) * (lev[t - 1] if t else 0.0)) / (m - 1)
               for t in range(p + 1)]
    mods, freq = [], []
    for a in range(3):
        f = np.fft.fftfreq(grid[a], 1.0 / grid[a])
        s = sum(lev[k + 1] * np.exp(2j * np.pi * np.arange(grid[a]) * k / grid[a])
                for k in range(p - 1))
        m = np.abs(s) ** 2
        for i in np.nonzero(m < 1e-7)[0]:
            m[i] = 0.5 * (m[i - 1] + m[(i + 1) % grid[a]])
        mods.append(torch.tensor(m, device=dev))
        freq.append(torch.tensor(f / float(box[a]), device=dev))
    m2 = (freq[0] ** 2)[:, None, None] + (freq[1] ** 2)[None, :, None] + (freq[2] ** 2)
    g = torch.exp(-math.pi ** 2 * m2 / beta ** 2) / (math.pi * float(box.prod()) * m2)
    g = g / (mods[0][:, None, None] * mods[1][None, :, None] * mods[2])
    g[0, 0, 0] = 0.0
    return g


_ORDERS = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (2, 0, 0), (1, 1, 0), (1, 0, 1),
           (0, 2, 0), (0, 1, 1), (0, 0, 2)]


def _weights(sp, k):
    return (sp[k[0]][:, 0, :, None, None] * sp[k[1]][:, 1, None, :, None]
            * sp[k[2]][:, 2, None, None, :])


class _Exact:
    """FP64 energies, fields and operator products of one system (or, for a
    batch, of all its clusters as one block-diagonal system)."""

    def __init__(self, case, seed):
        s = _system(case, seed)
        self.s, self.n = s, len(s["pos"])
        m = _method(case, s)
        self.x = _t(s["pos"])
        self.mol = _t(s["mol"], torch.long)
        sizes = s.get("sizes", np.array([self.n // 5]))
        self.seg = torch.repeat_interleave(torch.arange(len(sizes), device=DEV),
                                           _t(5 * sizes, torch.long))
        self.nseg = len(sizes)
        self.box = None if s["box"] is None else _t(s["box"])
        self.beta = m.get("beta")
        self.q = _t(s["q"])
        i6 = torch.tensor([[0, 1, 2], [1, 3, 4], [2, 4, 5]], device=DEV)
        self.d, self.th, self.al = _t(s["dip"]), _t(s["quad"])[:, i6], _t(s["alpha"])[:, i6]
        if case.get("frames"):
            r = self.frame(self.x)
            self.loc = (self.d, self.th, self.al)
            self.d, self.th, self.al = self.rotated(r)
        abar = self.al.diagonal(dim1=1, dim2=2).sum(1) / 3
        self.sv = torch.where(abar > 0, abar.clamp(min=1e-30) ** -0.5, torch.zeros_like(abar))
        self.pol = torch.nonzero(abar > 0).reshape(-1)
        self.ainv = torch.zeros_like(self.al)
        self.ainv[self.pol] = torch.linalg.inv(self.al[self.pol])
        self.ij = _pairs(self.x, self.box, m.get("cutoff"), self.seg)
        if self.box is not None:
            self.grid = m["grid"]
            self.infl = _influence(self.box, self.grid, m["order"], self.beta, DEV)
        self.op = None

    def frame(self, x):
        unit = lambda v: v / v.norm(dim=-1, keepdim=True)   # noqa: E731
        f = _t(self.s["frames"], torch.long)
        o, a, b = x[f[:, 0]], x[f[:, 1]], x[f[:, 2]]
        da, db = a - o, b - o
        if self.box is not None:
            da = da - self.box * torch.round(da.detach() / self.box)
            db = db - self.box * torch.round(db.detach() / self.box)
        u, v = unit(da), unit(db)
        ez = unit(u + v)
        ex = unit(u - (u * ez).sum(-1, keepdim=True) * ez)
        return torch.stack([ex, torch.linalg.cross(ez, ex), ez], -1)

    def rotated(self, r):
        d, th, al = self.loc
        rt = r.transpose(1, 2)
        return ((r @ d[:, :, None])[:, :, 0], r @ th @ rt, r @ al @ rt)

    # -- energy functional W(mu) and its gradients, pair chunk by pair chunk
    def real(self, x, d, th, mu, lo, hi):
        i, j = self.ij[0, lo:hi], self.ij[1, lo:hi]
        r = _separation(x, i, j, self.box)
        dist = r.norm(dim=1)
        e = _base(dist, self.beta, 4)
        bare = _base(dist, None, 4)
        tp = _thole(dist, self.sv[i], self.sv[j])
        same = (self.mol[i] == self.mol[j]) & (self.seg[i] == self.seg[j])
        inter = ~same
        perm = [(self.q[k], d[k], th[k]) for k in (i, j)]
        comb = [(self.q[k], d[k] + mu[k], th[k]) for k in (i, j)]
        z = torch.zeros_like(dist)
        ind = [(z, mu[k], torch.zeros_like(th[k])) for k in (i, j)]
        damp = [t * c * inter for t, c in zip(tp, bare)]
        # different molecules: E - damping for M' = (q, d + mu, Theta), the
        # undamped rest for the permanent pair; same molecule: E - bare for
        # M', the damped kernel between the induced dipoles
        c1 = [a - torch.where(same, b, g) for a, b, g in zip(e, bare, damp)]
        c2 = [(b - t * b) * same for b, t in zip(bare, tp)]
        c2[0], c2[3], c2[4] = z, z, z
        u = _interaction(c1, *comb, r) + _interaction(damp, *perm, r) + _interaction(c2, *ind, r)
        return u, self.seg[i]

    def recip(self, x, d, th, mu):
        idx, sp = _splines(x, self.box, self.grid, 5)
        dm = d + mu
        amp = [self.q, dm[:, 0], dm[:, 1], dm[:, 2], th[:, 0, 0] / 3, 2 * th[:, 0, 1] / 3,
               2 * th[:, 0, 2] / 3, th[:, 1, 1] / 3, 2 * th[:, 1, 2] / 3, th[:, 2, 2] / 3]
        val = sum(a[:, None, None, None] * _weights(sp, k) for a, k in zip(amp, _ORDERS))
        flat = self.flat(idx)
        grid = torch.zeros(self.infl.numel(), dtype=torch.float64, device=x.device)
        f = torch.fft.fftn(grid.index_add(0, flat, val.reshape(-1)).reshape(self.grid))
        b = self.beta
        selfe = (b / math.sqrt(math.pi) * self.q ** 2
                 + 2 * b ** 3 / (3 * math.sqrt(math.pi)) * (dm ** 2).sum(1)
                 + 8 * b ** 5 / (45 * math.sqrt(math.pi)) * (th ** 2).sum((1, 2))).sum()
        return 0.5 * (self.infl * (f.real ** 2 + f.imag ** 2)).sum() - selfe

    def flat(self, idx):
        return ((idx[:, 0, :, None, None] * self.grid[1] + idx[:, 1, None, :, None])
                * self.grid[2] + idx[:, 2, None, None, :]).reshape(-1)

    def functional(self, mu, forces):
        """Energies per segment without the polarization self energy, and
        the gradients with respect to x, d, Theta and mu."""
        leaves = [t.detach().clone().requires_grad_(k == 3 or forces)
                  for k, t in enumerate((self.x, self.d, self.th, mu))]
        e = torch.zeros(self.nseg, dtype=torch.float64, device=DEV)
        step = 2_000_000
        for lo in range(0, self.ij.shape[1], step):
            u, seg = self.real(*leaves, lo, min(lo + step, self.ij.shape[1]))
            u.sum().backward()
            e = e.index_add(0, seg, u.detach())
        if self.box is not None:
            u = self.recip(*leaves)
            u.backward()
            e = e + u.detach()
        zero = lambda t: torch.zeros_like(t) if t.grad is None else t.grad   # noqa: E731
        return e, [zero(t) for t in leaves]

    # -- the operator T
    def field_of(self, p):
        """Total field of dipoles p at the polarizable sites."""
        if self.op is None:
            k = (self.sv[self.ij[0]] > 0) & (self.sv[self.ij[1]] > 0)
            i, j = self.ij[:, k]
            r = _separation(self.x, i, j, self.box)
            dist = r.norm(dim=1)
            e, bare = _base(dist, self.beta, 2), _base(dist, None, 2)
            tp = _thole(dist, self.sv[i], self.sv[j])
            self.op = (i, j, r, e[1] - tp[1] * bare[1], e[2] - tp[2] * bare[2])
            if self.box is not None:
                xp = self.x[self.pol]
                idx, sp = _splines(xp, self.box, self.grid, 5)
                self.spline = (self.flat(idx), [_weights(sp, o) for o in _ORDERS[1:4]])
        i, j, r, c1, c2 = self.op
        f = torch.zeros_like(p)
        f.index_add_(0, i, (c2 * (r * p[j]).sum(1))[:, None] * r - c1[:, None] * p[j])
        f.index_add_(0, j, (c2 * (r * p[i]).sum(1))[:, None] * r - c1[:, None] * p[i])
        if self.box is not None:
            flat, w = self.spline
            pp = p[self.pol]
            val = sum(pp[:, a, None, None, None] * w[a] for a in range(3)).reshape(-1)
            g = torch.zeros(self.infl.numel(), dtype=torch.float64, device=DEV)
            g.index_add_(0, flat, val)
            phi = torch.fft.ifftn(torch.fft.fftn(g.reshape(self.grid)) * self.infl).real
            local = (phi.reshape(-1) * g.numel())[flat].reshape(w[0].shape)
            rec = torch.stack([(local * w[a]).sum((1, 2, 3)) for a in range(3)], 1)
            f[self.pol] += 4 * self.beta ** 3 / (3 * math.sqrt(math.pi)) * pp - rec
        return f

    def times_t(self, p):
        out = torch.zeros_like(p)
        t = (self.ainv @ p[:, :, None])[:, :, 0] - self.field_of(p)
        out[self.pol] = t[self.pol]
        return out

    def field(self):
        _, g = self.functional(torch.zeros_like(self.x), False)
        out = torch.zeros_like(self.x)
        out[self.pol] = -g[3][self.pol]
        return out

    def solve(self, e0, steps=None, omega=0.0):
        """Conjugate gradient from alpha E: to 1e-14 D, or `steps` steps and
        the peek step."""
        apply = lambda v: (self.al @ v[:, :, None])[:, :, 0]   # noqa: E731
        x = apply(e0)
        r = e0 - self.times_t(x)
        z = apply(r)
        p, rz = z, (r * z).sum()
        for k in range(steps or 100):
            if steps is None and DEBYE * math.sqrt(float((z * z).sum()) / len(self.pol)) < 1e-14:
                break
            tp = self.times_t(p)
            g = rz / (p * tp).sum()
            x, r = x + g * p, r - g * tp
            z = apply(r)
            new = (r * z).sum()
            p, rz = z + new / rz * p, new
        return x + omega * z


def exact(case, seed):
    e = _Exact(case, seed)
    kind = case["kind"]
    if kind == "matvec":
        p = torch.zeros_like(e.x)
        p[e.pol] = _t(e.s["p"])[e.pol]
        return dict(tp=e.times_t(p))
    e0 = e.field()
    if kind == "field":
        return dict(field=e0)
    mu = e.solve(e0, 2, 1.0) if kind == "tcg" else e.solve(e0)
    e_pol = torch.zeros(e.nseg, dtype=torch.float64, device=DEV)
    e_pol.index_add_(0, e.seg, -0.5 * COULOMB * (mu * e0).sum(1))
    if kind == "tcg":
        return dict(e_pol=float(e_pol), mu=mu)
    e_elec, _ = e.functional(torch.zeros_like(mu), False)
    _, g = e.functional(mu, True)
    grad = g[0]
    if case.get("frames"):
        x = e.x.detach().clone().requires_grad_(True)
        d, th, al = e.rotated(e.frame(x))
        # 1/2 mu alpha^-1 mu at fixed mu: -1/2 v alpha v with v = alpha^-1 mu
        v = (e.ainv @ mu[:, :, None])[:, :, 0]
        w = (d * g[1]).sum() + (th * g[2]).sum() - 0.5 * (v * (al @ v[:, :, None])[:, :, 0]).sum()
        grad = grad + torch.autograd.grad(w, x)[0]
    out = dict(e_pol=e_pol, e_elec=COULOMB * e_elec, forces=-COULOMB * grad, mu=mu)
    if kind != "batch":
        out.update(e_pol=float(out["e_pol"]), e_elec=float(out["e_elec"]))
    if case.get("frames"):
        out["virial"] = None
    return out
