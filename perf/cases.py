"""Timed cases of the ray tracer: what a program built on it has it do.

Each case is a dict of plain values.  ``prepare`` draws the octree of the
potential, the observers and the rays from a seed and builds the Grid and the
descriptors that a program keeps between calls; ``run`` is one call (or, for
the differentiated cases, one forward and backward) through the package's
public entry points with its output and workspace buffers kept; ``exact`` is
the same method in plain float64 torch.

    listed()               the cases
    draw(rng)              one more case of the same ranges
    prepare(case, seed)    the state one pass needs, on the GPU
    run(state)             one pass, its outputs
    work(case)             bytes and operations one pass cannot do without
    exact(case, seed)      the outputs in float64, or None

Lengths are in Mpc/h, c = 1.  Trees: a periodic Gaussian potential
(P(k) ~ k^-3, rms 1e-5) on the coarse grid, plus truncated NFW-like haloes and
refinement where the density is high on the AMR trees.
"""
import math
import types

import numpy as np
import torch

import paper_2111_08744_amd as M

COSMO = (0.3, 0.7, 0.7)
H0 = 1.0 / 2997.92458
DEV = "cuda"


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    uni = {"n0": 64, "box": 500.0, "levels": 0, "spc": 10, "order": 1}
    amr3 = {"n0": 64, "box": 500.0, "levels": 3, "haloes": 60, "spc": 4, "order": 1}
    amr5 = {"n0": 32, "box": 250.0, "levels": 5, "haloes": 40, "spc": 4, "order": 1}
    return [
        # a quick low-resolution sky (the uniform workload): few rays, so
        # latency counts
        {"name": "sky_3k", "kind": "cast", **uni, "rays": "sky", "nside": 16, "z": 0.5},
        # a lensing map of the whole sky on a uniform grid
        {"name": "sky_197k", "kind": "cast", **uni, "rays": "sky", "nside": 128, "z": 1.0},
        # many observers in one call, each with its own source redshift
        {"name": "cones_1m", "kind": "cast", **uni, "rays": "cones", "observers": 64, "nside": 128, "z": 2.0},
        # the AMR workload: the whole sky through 128^3 + 3 levels (about 1e7 cells)
        {"name": "amr_sky_786k", "kind": "cast", **amr3, "n0": 128, "haloes": 200, "rays": "sky", "nside": 256,
         "z": 1.0},
        # a catalogue's directions through a deep tree, an odd number of them
        {"name": "amr_dirs_5k", "kind": "cast", **amr5, "rays": "dirs", "count": 5003, "z": 0.5},
        # third-order (TSC) interpolation
        {"name": "tsc_49k", "kind": "cast", **uni, "order": 2, "rays": "sky", "nside": 64, "z": 1.0},
        # distortion matrices of a sky by forward-mode tangents
        {"name": "jacobian_amr_49k", "kind": "jacobian", **amr3, "rays": "sky", "nside": 64, "z": 1.0},
        # the paper's infinitesimal beam, and the convergence and shear maps from it
        {"name": "beam_49k", "kind": "beam", **uni, "rays": "sky", "nside": 64, "z": 1.0},
        # the differentiated workload: distortion matrix and cell gradient by the reverse sweep
        {"name": "adjoint_131k", "kind": "adjoint", **uni, "rays": "pixels", "nside": 512, "first": 0,
         "count": 131072, "z": 1.0, "ckpt": 32},
        # one training step of a potential through torch.autograd on a deep tree
        {"name": "train_amr_12k", "kind": "train", **amr5, "rays": "sky", "nside": 32, "z": 0.5, "ckpt": 32},
        # a relativistic catalogue: the geodesics to given sources
        {"name": "finder_4k", "kind": "finder", **uni, "count": 4096, "chi": 1500.0},
        # lensing maps of a high-resolution sky's matrices
        {"name": "maps_12m", "kind": "maps", "count": 12 * 1024 * 1024},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """A case of the listed ones' ranges: any kind, any size between its
    smallest and largest call."""
    kind = rng.choice(["cast", "cast", "cast", "tsc", "jacobian", "beam", "adjoint", "train", "finder", "maps"])
    if kind == "maps":
        return {"kind": kind, "count": int(_log(rng, 1e3, 12e6))}
    amr = kind == "train" or (kind in ("cast", "tsc", "jacobian") and rng.random() < 0.5)
    if not amr:
        c = {"n0": rng.choice([32, 64]), "levels": 0, "spc": rng.randint(6, 10)}
    elif rng.random() < 0.5:
        c = {"n0": 64, "levels": 3, "haloes": rng.randint(30, 70), "spc": rng.randint(3, 5)}
    else:
        c = {"n0": 32, "levels": 5, "haloes": rng.randint(20, 50), "spc": rng.randint(3, 5)}
    c = {"kind": "cast" if kind == "tsc" else kind, "box": c["n0"] * 7.8125, **c, "order": 2 if kind == "tsc" else 1}
    if kind == "finder":
        return {**c, "count": int(_log(rng, 100, 4096)), "chi": round(rng.uniform(400.0, 1500.0), 1)}
    most = {"cast": 600e3, "tsc": 60e3, "jacobian": 100e3, "beam": 50e3, "adjoint": 100e3, "train": 12e3}[kind]
    count = int(_log(rng, 200, most))
    c["z"] = round(rng.uniform(0.1, 1.0 if kind != "train" else 0.5), 3)
    if kind == "cast" and rng.random() < 0.3:
        nside = rng.choice([8, 16, 32, 64])
        c.update(rays="cones", observers=min(64, max(2, count // nside ** 2)), nside=nside)
    elif rng.random() < 0.5:
        c.update(rays="dirs", count=count)
    else:
        nside = 1 << rng.randint(max(2, math.ceil(math.log2(math.sqrt(count / 12.0)))), 10)
        c.update(rays="pixels", nside=nside, first=rng.randint(0, 12 * nside * nside - count), count=count)
    if kind in ("adjoint", "train"):
        c["ckpt"] = rng.choice([16, 32, 64])
    return c


# ---------------------------------------------------------------------------
# Inputs: the tree, the observers and the rays
# ---------------------------------------------------------------------------
def _rng(seed, stream):
    return np.random.Generator(np.random.PCG64([int(seed), stream]))


def _gaussian(n, box, seed):
    """Periodic Gaussian potential, P(k) ~ k^-3, rms 1e-5, and its central differences."""
    white = torch.from_numpy(_rng(seed, 1).standard_normal((n, n, n), dtype=np.float32)).to(DEV).double()
    k = 2 * math.pi * torch.fft.fftfreq(n, d=box / n, device=DEV, dtype=torch.float64)
    kz = 2 * math.pi * torch.fft.rfftfreq(n, d=box / n, device=DEV, dtype=torch.float64)
    k2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + kz[None, None, :] ** 2
    k2[0, 0, 0] = 1.0
    amp = k2 ** -0.75
    amp[0, 0, 0] = 0.0
    phi = torch.fft.irfftn(torch.fft.rfftn(white) * amp, s=(n, n, n))
    phi = phi * (1e-5 / phi.square().mean().sqrt())
    g = torch.stack([(phi.roll(-1, d) - phi.roll(1, d)) / (2 * box / n) for d in range(3)], -1)
    return phi, g


def _sample(grid, x, box):
    """Trilinear sample of a periodic cell-centred grid [n, n, n, q] at x [m, 3]."""
    n = grid.shape[0]
    u = x / (box / n) - 0.5
    b = u.floor()
    t = u - b
    b = b.long()
    out = 0.0
    for o in range(8):
        c = [(b[:, d] + ((o >> d) & 1)) % n for d in range(3)]
        w = math.prod(t[:, d] if (o >> d) & 1 else 1 - t[:, d] for d in range(3))
        out = out + w[:, None] * grid[c[0], c[1], c[2]]
    return out


def _tree(case, seed):
    """The cells, level by level: ijk [m_l, 3] of every level, and (phi, gx, gy,
    gz) of all of them as float32 [n, 4]."""
    n, box, levels = case["n0"], case["box"], case["levels"]
    phi, g = _gaussian(n, box, seed)
    a = torch.arange(n, device=DEV)
    ijk = [torch.stack(torch.meshgrid(a, a, a, indexing="ij"), -1).reshape(-1, 3)]
    vals = [torch.cat([phi.reshape(-1, 1), g.reshape(-1, 3)], 1)]
    if levels:
        m = case["haloes"]
        r = _rng(m, 2)             # the haloes, and with them the cells, are the case's; the values the seed's
        pos = r.uniform(0, box, (m, 3))
        p0 = np.exp(r.uniform(math.log(1e-6), math.log(3e-5), m))
        rs = np.exp(r.uniform(math.log(0.2), math.log(1.5), m))
        d0 = (1e9 if levels <= 3 else 3e8) * p0 / rs ** 2
        threshold = 8.0 if levels <= 3 else 30.0
        field = torch.cat([phi[..., None], g], -1)

        def near(x, h):
            d = x - torch.tensor(pos[h], device=DEV)
            return d - box * (d / box).round()

        for lev in range(levels):
            half = 0.5 * box / (n << lev)
            x = (ijk[-1].double() + 0.5) * (2 * half)
            rho = torch.ones(len(x), device=DEV, dtype=torch.float64)
            for h in range(m):   # at the point of the cell nearest to the halo
                rr = (near(x, h).abs() - half).clamp(min=0.0).square().sum(1).sqrt()
                y = (rr / rs[h]).clamp(min=1e-3)
                rho += torch.where(rr < 25 * rs[h], d0[h] / (y * (1 + y) ** 2), 0.0)
            par = ijk[-1][rho > threshold]
            if not len(par):
                break
            octs = torch.tensor([[o & 1, (o >> 1) & 1, o >> 2] for o in range(8)], device=DEV)
            ijk.append((2 * par[:, None, :] + octs).reshape(-1, 3))
            vals.append(_sample(field, (ijk[-1].double() + 0.5) * half, box))
        p0 = p0 * _rng(seed, 2).uniform(0.7, 1.3, m)
        for lev, v in enumerate(vals):
            x = (ijk[lev].double() + 0.5) * (box / (n << lev))
            for h in range(m):
                d = near(x, h)
                rr = d.square().sum(1).sqrt()
                y = (rr / rs[h]).clamp(min=1e-12)
                f, ins = torch.log1p(y) / y, rr < 25 * rs[h]
                v[:, 0] -= torch.where(ins, p0[h] * (f - math.log1p(25.0) / 25.0), 0.0)
                fr = -p0[h] * (1 / (y * (1 + y)) - f / y) / rs[h] / rr.clamp(min=1e-12)
                v[:, 1:] += torch.where(ins, fr, 0.0)[:, None] * d
    return ijk, torch.cat(vals).float()


def _rays(case, seed):
    """Observers [m, 3], stops [m] (redshift), and the ray arguments of CastConfig."""
    r = _rng(seed, 3)
    box = case["box"]
    centre = np.full((1, 3), 0.5 * box)
    kind = case["rays"]
    if kind == "cones":      # one NESTED base pixel per observer
        m, ns = case["observers"], case["nside"]
        obs = r.uniform(0, box, (m, 3))
        z = r.uniform(0.1, max(0.1001, case["z"]), m)
        return obs, z, {"nside": ns, "pix_first": r.integers(0, 12, m) * ns * ns, "pix_count": np.full(m, ns * ns)}
    z = np.array([case["z"]])
    if kind == "sky":
        return centre, z, {"nside": case["nside"]}
    if kind == "pixels":
        return centre, z, {"nside": case["nside"], "pix_first": [case["first"]], "pix_count": [case["count"]]}
    v = r.standard_normal((case["count"], 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    return centre, z, {"nside": 1, "pix_count": [case["count"]], "dirs": torch.from_numpy(v).to(DEV)}


def _sources(case, seed):
    r = _rng(seed, 4)
    v = r.standard_normal((case["count"], 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    obs = np.full(3, 0.5 * case["box"])
    return obs, obs + v * r.uniform(200.0, case["chi"], case["count"])[:, None]


def _matrices(case, seed):
    """Distortion matrices of weak lensing: convergence and shear of a few per
    cent, a rotation a hundred times smaller."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    k, g1, g2, w = 0.02 * torch.randn((4, case["count"]), generator=g, device=DEV, dtype=torch.float64)
    w = 0.01 * w
    return torch.stack([1 - k - g1, -g2 - w, -g2 + w, 1 - k + g1], 1).reshape(-1, 2, 2).float()


def prepare(case, seed):
    s = types.SimpleNamespace(case=case, kind=case["kind"], ws=None, out=None)
    if s.kind == "maps":
        s.A = _matrices(case, seed)
        return s
    ijk, vals = _tree(case, seed)
    level = torch.cat([torch.full((len(c),), i, dtype=torch.uint8, device=DEV) for i, c in enumerate(ijk)])
    host = vals.cpu().numpy()
    cells = types.SimpleNamespace(box=case["box"], n0=case["n0"], max_level=len(ijk) - 1, periodic=True,
                                  level=level.cpu().numpy(), ijk=torch.cat(ijk).int().cpu().numpy(),
                                  phi=np.ascontiguousarray(host[:, 0]), grad=np.ascontiguousarray(host[:, 1:]))
    del ijk
    s.grid = M.Grid(cells, COSMO, device=DEV)
    adaptive = case["levels"] > 0
    if s.kind == "finder":
        s.obs, s.src = _sources(case, seed)
        return s
    obs, z, rays = _rays(case, seed)
    s.cfg = M.CastConfig(obs, z, steps_per_cell=case["spc"], adaptive=adaptive, order=case["order"],
                         checkpoint_every=case.get("ckpt", 0), **rays)
    n = s.cfg.n_rays()
    s.out = M.alloc_outputs(n, DEV)
    if s.kind == "adjoint":     # the cotangents of a fit to observed deflections and redshifts
        g = torch.Generator(device=DEV).manual_seed(int(seed))
        s.g_alpha = torch.randn((n, 2), generator=g, device=DEV)
        s.g_z = torch.randn((n,), generator=g, device=DEV, dtype=torch.float64)
    if s.kind == "train":
        s.values = vals.requires_grad_()
        g = torch.Generator(device=DEV).manual_seed(int(seed))
        s.target = 1e-5 * torch.randn((n, 2), generator=g, device=DEV)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _public(d):
    return {k: v for k, v in d.items() if not k.startswith("_")}


def run(s):
    if s.kind == "maps":
        return M.lensing_maps(s.A)
    if s.kind == "finder":
        res = M.find_geodesics(s.grid, s.obs, s.src, steps_per_cell=s.case["spc"], tol=1e-9, ws=s.ws)
        s.ws = res["_ws"]
        return _public(res)
    if s.kind == "cast":
        return _public(M.cast(s.grid, s.cfg, s.out, s.out.get("_ws")))
    if s.kind == "jacobian":
        return _public(M.jacobian(s.grid, s.cfg, s.out, s.out.get("_ws")))
    if s.kind == "beam":
        out = M.infinitesimal_beam(s.grid, s.cfg, s.out, s.out.get("_ws"))
        return {**_public(out), "maps": M.lensing_maps(out["A"])}
    if s.kind == "adjoint":
        out = M.cast(s.grid, s.cfg, s.out, s.out.get("_ws"))
        res = M.adjoint(s.grid, s.cfg, out, dL_dalpha=s.g_alpha, dL_dz=s.g_z, jacobian=True, cells=True, ws=s.ws)
        s.ws = res["_ws"]
        return {"cast": _public(out), "adjoint": _public(res)}
    alpha, z5 = M.cast_differentiable(s.values, s.grid, s.cfg)
    loss = (alpha - s.target).square().sum()
    grad, = torch.autograd.grad(loss, s.values)
    return {"alpha": alpha, "z5": z5, "grad": grad}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _chi(z):
    """Comoving distance to z."""
    a, w = np.polynomial.legendre.leggauss(64)
    x = 0.5 * z * (a + 1)
    return float(0.5 * z * np.sum(w / (H0 * np.sqrt(COSMO[0] * (1 + x) ** 3 + COSMO[1]))))


def _count(case):
    if case["rays"] == "sky":
        return 12 * case["nside"] ** 2
    if case["rays"] == "cones":
        return case["observers"] * case["nside"] ** 2
    return case["count"]


# operations of an RK4 step with CIC (8 corners, 4 fields, 4 stages and the
# right-hand sides), with TSC (27 corners), with two tangents, with six more
# gradient samples, and of a step's reverse (two recomputations of the step
# and three columns through the transposed stages)
STEP_FLOPS = {"cast": 580, "tsc": 1300, "jacobian": 1700, "beam": 1100, "adjoint": 580 + 3500, "train": 580 + 2200}


def work(case):
    kind = case["kind"]
    if kind == "maps":
        return {"bytes": 36.0 * case["count"], "flops": 60.0 * case["count"]}
    cells = 16.0 * case["n0"] ** 3
    step = case["box"] / case["n0"] / case["spc"]
    if kind == "finder":
        steps = case["count"] * 0.5 * (200.0 + case["chi"]) / step
        # four plain casts, one cast with its matrix
        return {"bytes": cells + 100.0 * case["count"], "flops": steps * (4 * 580 + 1700)}
    n = _count(case)
    chi = _chi(case["z"]) if case["rays"] != "cones" else 0.5 * (_chi(0.1) + _chi(max(0.1001, case["z"])))
    per = STEP_FLOPS["tsc" if case["order"] == 2 else kind]
    grads = {"adjoint": 1.0, "train": 2.0}.get(kind, 0.0)    # cell gradients written, values read
    return {"bytes": (1 + grads) * cells + n * (24.0 + 88.0), "flops": n * chi / step * per}


# ---------------------------------------------------------------------------
# The method in float64
# ---------------------------------------------------------------------------
class _Background:
    """a'/a on a dense table of conformal time (cubic Hermite)."""

    def __init__(self, n=16384):
        gx, gw = np.polynomial.legendre.leggauss(20)
        om, ol = COSMO[:2]

        def speed(y):                 # d eta / d sqrt(a)
            return 2.0 / (H0 * np.sqrt(om + ol * y ** 6))

        def eta(y):
            y = np.atleast_1d(y)
            c = (np.arange(8) + 0.5) / 8
            at = y[:, None, None] * (c[:, None] + gx / 16)
            return (y[:, None, None] / 16 * gw * speed(at)).sum((1, 2))

        self.eta_of_a = lambda a: float(eta(math.sqrt(a))[0])
        self.eta0 = self.eta_of_a(1.0)
        self.lo = self.eta_of_a(1 / 4.0)
        self.dx = (self.eta0 + 50.0 - self.lo) / (n - 1)
        e = self.lo + self.dx * np.arange(n)
        y = np.linspace(0.5, 1.01, n)
        y = np.interp(e, eta(y), y)
        for _ in range(6):
            y -= (eta(y) - e) / speed(y)
        a = y * y
        s = np.sqrt(om / a + ol * a * a)
        H = H0 * s
        dH = H0 * (-om / a ** 2 + 2 * ol * a) / (2 * s) * a * H
        c0, c1 = H[:-1], self.dx * dH[:-1]
        c2 = 3 * np.diff(H) - self.dx * (2 * dH[:-1] + dH[1:])
        c3 = -2 * np.diff(H) + self.dx * (dH[:-1] + dH[1:])
        self.c = torch.from_numpy(np.stack([c0, c1, c2, c3], 1)).to(DEV)

    def __call__(self, eta):
        """a'/a and its derivative at eta [m]."""
        u = (eta - self.lo) / self.dx
        i = u.floor().long().clamp(0, self.c.shape[0] - 1)
        t = u - i
        c = self.c[i]
        return (c[:, 0] + t * (c[:, 1] + t * (c[:, 2] + t * c[:, 3])),
                (c[:, 1] + t * (2 * c[:, 2] + 3 * t * c[:, 3])) / self.dx)


class _Field:
    """(phi, gx, gy, gz) by CIC or TSC at the finest level, not above the
    leaf's, at which the whole stencil exists."""

    def __init__(self, case, ijk, vals):
        self.n0, self.box, self.order = case["n0"], case["box"], case["order"]
        self.vals = vals.double()
        o = [0, 1] if self.order == 1 else [-1, 0, 1]
        self.off = torch.tensor([[i, j, k] for i in o for j in o for k in o], device=DEV)
        ids, whole, start, self.base = [], [], 0, []
        for lev, c in enumerate(ijk):
            m = self.n0 << lev
            t = torch.full((m * m * m,), -1, dtype=torch.int32, device=DEV)
            t[self.flat(c, m)] = torch.arange(start, start + len(c), dtype=torch.int32, device=DEV)
            e = (t >= 0).reshape(m, m, m)
            w = e
            for d in range(3):
                w = torch.stack([w.roll(-s, d) for s in o]).all(0)
            self.base.append(sum(len(x) for x in ids))
            ids.append(t)
            whole.append(w.reshape(-1))
            start += len(c)
        self.ids, self.whole = torch.cat(ids), torch.cat(whole)
        self.top = len(ijk) - 1

    @staticmethod
    def flat(c, m):
        c = c.long() & (m - 1)
        return (c[..., 0] * m + c[..., 1]) * m + c[..., 2]

    def leaf(self, x):
        lev = torch.zeros(len(x), dtype=torch.int64, device=DEV)
        for s in range(1, self.top + 1):
            m = self.n0 << s
            lev = torch.where(self.ids[self.base[s] + self.flat((x * (m / self.box)).floor(), m)] >= 0, s, lev)
        return lev

    def __call__(self, x, jac=False):
        """Values [m, 4] at x [m, 3]; with jac also their derivatives [m, 4, 3]."""
        lev = self.leaf(x) if self.top else None
        for s in range(self.top + 1):
            m = self.n0 << s
            u = x * (m / self.box) - (0.5 if self.order == 1 else 0.0)
            bs = u.floor()
            here = (self.base[s] + self.flat(bs, m))
            if s == 0:
                t, at = u - bs, self.flat(bs[:, None, :].long() + self.off, m)
                h = torch.full((len(x),), self.box / m, device=DEV, dtype=torch.float64)
            else:
                ok = self.whole[here] & (lev >= s)
                t = torch.where(ok[:, None], u - bs, t)
                at = torch.where(ok[:, None], self.base[s] + self.flat(bs[:, None, :].long() + self.off, m), at)
                h = torch.where(ok, self.box / m, h)
        v = self.vals[self.ids[at].long()]                        # [m, q, 4]
        if self.order == 1:
            w1, d1 = torch.stack([1 - t, t], 2), torch.stack([-torch.ones_like(t), torch.ones_like(t)], 2)
        else:
            w1 = torch.stack([0.5 * (1 - t) ** 2, 0.75 - (t - 0.5) ** 2, 0.5 * t ** 2], 2)
        def outer(a, b, c):
            return (a[:, :, None, None] * b[:, None, :, None] * c[:, None, None, :]).reshape(len(x), 1, -1)
        f = (outer(w1[:, 0], w1[:, 1], w1[:, 2]) @ v)[:, 0]
        if not jac:
            return f
        ws = [[d1[:, d] if d == e else w1[:, d] for d in range(3)] for e in range(3)]
        return f, torch.cat([outer(*w) @ v for w in ws], 1).transpose(1, 2) / h[:, None, None]


def _screen(v):
    """e_phi and -e_theta at directions v [m, 3], stacked [m, 2, 3]."""
    rho = v[:, :2].norm(dim=1)
    r = v.norm(dim=1)
    cp, sp, ct, st = v[:, 0] / rho, v[:, 1] / rho, v[:, 2] / r, rho / r
    return torch.stack([torch.stack([-sp, cp, 0 * sp], 1), torch.stack([-cp * ct, -sp * ct, st], 1)], 1)


class _Tracer:
    """RK4 on (eta, x, k0, k) [m, 8], optionally with two tangents [m, 2, 8] or
    the infinitesimal beam's sums, from one observer to one redshift."""

    def __init__(self, case, ijk, vals):
        self.F, self.bg = _Field(case, ijk, vals), _Background()
        self.h0, self.spc, self.adaptive = case["box"] / case["n0"], case["spc"], case["levels"] > 0

    def rhs(self, y, dy=None):
        H, dH = self.bg(y[:, 0])
        got = self.F(y[:, 1:4], jac=dy is not None)
        G = (got if dy is None else got[0])[:, 1:]
        k0, k = y[:, 4:5], y[:, 5:]
        H = H[:, None]
        psi = (G * k).sum(1, keepdim=True)
        f = torch.cat([k0, k, -2 * H * k0 ** 2 - 2 * psi * k0, -2 * H * k0 * k + 2 * psi * k - 2 * G * k0 ** 2], 1)
        if dy is None:
            return f, None
        dG = (got[1][:, None, 1:] @ dy[:, :, 1:4, None])[..., 0]
        k0, k, H, psi, G = (q[:, None] for q in (k0, k, H, psi, G))
        dh = dH[:, None, None] * dy[:, :, :1]
        d0, dk = dy[:, :, 4:5], dy[:, :, 5:]
        dpsi = (dG * k + G * dk).sum(2, keepdim=True)
        df = torch.cat([d0, dk, -2 * dh * k0 ** 2 - 4 * H * k0 * d0 - 2 * dpsi * k0 - 2 * psi * d0,
                        -2 * dh * k0 * k - 2 * H * (d0 * k + k0 * dk) + 2 * dpsi * k + 2 * psi * dk
                        - 2 * dG * k0 ** 2 - 4 * G * k0 * d0], 2)
        return f, df

    def step(self, y, dl, dy=None, ddl=None):
        dl = dl[:, None]
        fs, ds = 0.0, 0.0
        f = df = None
        for c, w in ((0.0, 1.0), (0.5, 2.0), (0.5, 2.0), (1.0, 1.0)):
            Y = y if f is None else y + c * dl * f
            dY = dy if dy is None or f is None else dy + c * (ddl[:, :, None] * f[:, None] + dl[:, None] * df)
            f, df = self.rhs(Y, dY)
            fs = fs + w * f
            if dy is not None:
                ds = ds + w * df
        out = y + dl / 6 * fs
        return out, None if dy is None else dy + (ddl[:, :, None] * fs[:, None] + dl[:, None] * ds) / 6

    def beam(self, y, o, lev):
        """Trace sample of the infinitesimal beam: chi and (T11, T12, T22)."""
        x, r = y[:, 1:4], y[:, 1:4] - o.x
        chi = r.norm(dim=1)
        e = _screen(torch.where(chi[:, None] > 0, r, o.n[o.idx]))
        h = (self.h0 / 2.0 ** lev)[:, None]
        rows = []
        for d in range(3):
            s = torch.zeros(3, device=DEV, dtype=torch.float64)
            s[d] = 1.0
            rows.append((self.F(x + h * s)[:, 1:] - self.F(x - h * s)[:, 1:]) / (2 * h))
        Hs = torch.stack(rows, 1)
        T = e @ (0.5 * (Hs + Hs.transpose(1, 2))) @ e.transpose(1, 2)
        return chi, torch.stack([T[:, 0, 0], T[:, 0, 1], T[:, 1, 1]], 1)

    def trace(self, obs, z, n, tangents=False, beam=False):
        """Casts n [m, 3] from obs [3]; a dict of the end states."""
        m = len(n)
        o = types.SimpleNamespace(x=torch.tensor(obs, device=DEV), n=n, idx=torch.arange(m, device=DEV))
        eta_s = self.bg.eta_of_a(1 / (1 + z))
        phi_o = self.F(o.x[None])[0, 0]
        kmag = ((1 + 2 * phi_o) / (1 - 2 * phi_o)).sqrt()
        y = torch.zeros((m, 8), device=DEV, dtype=torch.float64)
        y[:, 0], y[:, 1:4], y[:, 4], y[:, 5:] = self.bg.eta0, o.x, -1.0, kmag * n
        dy = None
        if tangents:
            dy = torch.zeros((m, 2, 8), device=DEV, dtype=torch.float64)
            dy[:, :, 5:] = kmag * _screen(n)
        land = [torch.empty_like(y), None if dy is None else torch.empty_like(dy)]
        sums = torch.zeros((m, 3, 2), device=DEV, dtype=torch.float64)       # trapezoids of chi T, chi^2 T
        prev = torch.zeros((m, 4), device=DEV, dtype=torch.float64)
        first = True
        while len(o.idx):
            lev = self.F.leaf(y[:, 1:4]) if self.adaptive or beam else 0
            if beam:
                chi, T = self.beam(y, o, lev)
                if not first:
                    self._trapezoid(sums, prev, o.idx, chi, T)
                prev[o.idx] = torch.cat([chi[:, None], T], 1)
                first = False
            ds = self.h0 / self.spc / (2.0 ** lev if self.adaptive else 1.0)
            dl = ds / -y[:, 4]
            stop = y[:, 0] + y[:, 4] * dl < eta_s
            if stop.any():
                land[0][o.idx[stop]] = y[stop]
                if tangents:
                    land[1][o.idx[stop]] = dy[stop]
                on = ~stop
                o.idx, y, dl = o.idx[on], y[on], dl[on]
                dy = dy[on] if tangents else None
                if not len(o.idx):
                    break
            ddl = dl[:, None] * dy[:, :, 4] / -y[:, 4:5] if tangents else None
            y, dy = self.step(y, dl, dy, ddl)
        y, dy = land
        dl = (y[:, 0] - eta_s) / -y[:, 4]
        for _ in range(2):
            e, _d = self.step(y, dl)
            dl = dl + (e[:, 0] - eta_s) / -e[:, 4]
        y, dy = self.step(y, dl, dy, torch.zeros((m, 2), device=DEV, dtype=torch.float64) if tangents else None)
        if beam:
            o.idx = torch.arange(m, device=DEV)
            chi, T = self.beam(y, o, self.F.leaf(y[:, 1:4]))
            self._trapezoid(sums, prev, o.idx, chi, T)
            I = sums[:, :, 0] - sums[:, :, 1] / chi[:, None]
            beam = torch.stack([1 - 2 * I[:, 0], -2 * I[:, 1], -2 * I[:, 1], 1 - 2 * I[:, 2]], 1).reshape(-1, 2, 2)
        return self.observables(o.x, n, z, phi_o, y, dy), beam

    @staticmethod
    def _trapezoid(sums, prev, idx, chi, T):
        c0, T0, c1 = prev[idx, :1], prev[idx, 1:], chi[:, None]
        w = 0.5 * (c1 - c0)
        sums[idx] += torch.stack([w * (c0 * T0 + c1 * T), w * (c0 ** 2 * T0 + c1 ** 2 * T)], 2)

    def observables(self, xo, n, z, phi_o, y, dy):
        r = y[:, 1:4] - xo
        chi = r.norm(dim=1)
        a_s, z0, K = 1 / (1 + z), z, -y[:, 4]
        f, jf = self.F(y[:, 1:4], jac=True) if dy is not None else (self.F(y[:, 1:4]), None)
        phi = f[:, 0]
        rh = r / chi[:, None]
        c = (rh * n).sum(1, keepdim=True)
        t = rh - c * n
        st = t.norm(dim=1)
        fac = torch.where(st > 0, -torch.atan2(st, c[:, 0]) / st, 0.0)
        z1 = z0 + (1 + z0) * (phi_o - phi)
        out = {"beta": torch.stack([torch.atan2(r[:, :2].norm(dim=1), r[:, 2]), torch.atan2(r[:, 1], r[:, 0])], 1),
               "alpha": fac[:, None] * (_screen(n) @ t[:, :, None])[..., 0],
               "z5": a_s * K * (1 + phi) / (1 + phi_o) - 1, "z0": torch.full_like(chi, z0), "phi_src": phi,
               "n_steps": None, "status": None, "hash": None, "chi": chi, "z1": z1, "z4": z1,
               "isw": torch.zeros_like(chi)}
        if dy is not None:
            flow, _ = self.rhs(y)
            dy = dy - flow[:, None] * (dy[:, :, :1] / flow[:, None, :1])
            out["jac"] = (_screen(r) @ dy[:, :, 1:4].transpose(1, 2)) / chi[:, None, None]
            out["dz_dtheta"] = a_s / (1 + phi_o) * (-dy[:, :, 4] * (1 + phi)[:, None] +
                                                    K[:, None] * (jf[:, None, 0] * dy[:, :, 1:4]).sum(2))
        return out


def _maps(A):
    A = A.double()
    a, b, c, d = A[:, 0, 0], A[:, 0, 1], A[:, 1, 0], A[:, 1, 1]
    r = torch.hypot(a + d, c - b)
    co, si = (a + d) / r, (c - b) / r
    s11, s12, s21, s22 = co * a + si * c, co * b + si * d, co * c - si * a, co * d - si * b
    return torch.stack([1 - 0.5 * r, 0.5 * (s22 - s11), -0.5 * (s12 + s21), torch.atan2(c - b, a + d),
                        1 / (a * d - b * c)], 1)


def _directions(rays):
    """NESTED pixel centres (Gorski et al. 2005), or the caller's directions."""
    if "dirs" in rays:
        return rays["dirs"]
    ns = rays["nside"]
    first = int(np.atleast_1d(rays.get("pix_first", 0))[0])
    count = int(np.atleast_1d(rays.get("pix_count", 12 * ns * ns))[0])
    p = np.arange(first, first + count)
    face, ip = p // (ns * ns), p % (ns * ns)
    x, y = np.zeros_like(p), np.zeros_like(p)
    for b in range(14):
        x |= ((ip >> (2 * b)) & 1) << b
        y |= ((ip >> (2 * b + 1)) & 1) << b
    ring = (2 + face // 4) * ns - x - y - 1
    nr = np.where(ring < ns, ring, np.where(ring > 3 * ns, 4 * ns - ring, ns))
    cap = nr ** 2 / (3.0 * ns * ns)
    zc = np.where(ring < ns, 1 - cap, np.where(ring > 3 * ns, cap - 1, (2 * ns - ring) * 2.0 / (3.0 * ns)))
    st = np.where((ring < ns) | (ring > 3 * ns), np.sqrt(cap * (2 - cap)), np.sqrt((1 - zc) * (1 + zc)))
    ph = 0.25 * np.pi * (2 * (face % 4) + (face // 4 != 1) + (x - y) / nr)
    return torch.from_numpy(np.stack([st * np.cos(ph), st * np.sin(ph), zc], 1)).to(DEV)


def exact(case, seed):
    kind = case["kind"]
    if kind == "maps":
        return _maps(_matrices(case, seed))
    # the finder's roots, many observers and millions of points take too long
    if kind == "finder" or case["rays"] == "cones" or case["n0"] << case["levels"] > 1024:
        return None
    n = _count(case)
    # about 10 us an operation for 2e5 rays, 5 us for few; some 100 a stage and
    # 40 for every level, twice that with tangents
    ops = 4 * (100 + 40 * case["levels"]) * {"jacobian": 2.0, "adjoint": 2.0, "beam": 2.5}.get(kind, 1.0)
    steps = _chi(case["z"]) / (case["box"] / case["n0"] / case["spc"]) * (1.5 if case["levels"] else 1.0)
    if ops * steps * (5e-6 + 3e-11 * n * (4 if case["order"] == 2 else 1)) > 40.0:
        return None
    ijk, vals = _tree(case, seed)
    tr = _Tracer(case, ijk, vals)
    obs, z, rays = _rays(case, seed)
    out, beam = tr.trace(obs[0], float(z[0]), _directions(rays), tangents=kind in ("jacobian", "adjoint"),
                         beam=kind == "beam")
    if kind == "beam":
        return {**out, "A": beam, "maps": _maps(beam)}
    if kind == "adjoint":
        jac, dz = out.pop("jac"), out.pop("dz_dtheta")
        return {"cast": out, "adjoint": {"jac": jac, "dz_dtheta": dz, "dL_dvalues": None, "ray_status": None}}
    if kind == "train":      # the cell gradient would take a reverse sweep of the whole path
        return {"alpha": out["alpha"], "z5": out["z5"], "grad": None}
    return out
