"""Performance cases of the CFNEB library: what a user's program has it do, through the
public entry points of paper_2510_16721_amd.cfneb, over the sizes it is used at.

Kinds of pass:
  step     a band in hand takes `steps` band steps, then its energies are read (a
           relaxation loop that looks at its band now and then); with the coordinates
           of every image, in the workspace that the program owns
  batch    the same for a batch of mixed bands
  relax    one structure is relaxed for `steps` steps from host arrays (band endpoints)
  request  a band is made from host arrays, displaced by the interior noise, stepped,
           read out (energies, the middle image) and released, as for one served request
  profile  the energy profile of a band at its coordinates: every image evaluated afresh

Results of FP32 bands (FP32 pair and three-body arithmetic) are returned in FP32, those
of FP64 bands in FP64; the force norm and the normalized arc length of FP32 hops are left
out, which close to the crystal are made of the rounding of FP32 forces.  The inputs are LJ FCC and diamond vacancy hops whose interior
images are displaced by seeded Gaussian noise, and graphite to diamond-like bands whose
endpoints are.
"""
import math

import numpy as np
import torch

from paper_2510_16721_amd import cfneb

GPA = 160.21766208  # eV / A^3 in GPa
FCC = np.array([[0.0, 0.0, 0.0], [0.0, 0.5, 0.5], [0.5, 0.0, 0.5], [0.5, 0.5, 0.0]])
STRESS = (60.0, -20.0, 10.0, 15.0, 0.0, -25.0)  # an applied non-hydrostatic load, GPa

DEFAULT = dict(kind="step", lattice="fcc", nx=4, ny=4, nz=4, images=7, steps=32, fp64=False,
               cell_filter=2, pressure=0.0, stress=False, climb=-1, refine=0, samples=0)


def _case(name=None, **kw):
    c = dict(DEFAULT, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # smallest calls: the 255-atom LJ vacancy hop in FP64 with its climbing image (the larger bands
        # start from endpoints that are not relaxed, where an image has no saddle to climb to)
        _case("lj_255_fp64_step", fp64=True, climb=50),
        # an ordinary LJ band, FP32, ragged against every tile size
        _case("lj_2047_step", nx=8, ny=8, nz=8, images=9),
        # an ordinary small Tersoff band
        _case("ts_511_step", lattice="diamond", nx=4, ny=4, nz=4, images=9),
        # a small band under an applied stress with the D-variant filter, FP64
        _case("ts_1727_fp64_stress_step", lattice="diamond", nx=6, ny=6, nz=6, images=9, fp64=True,
              cell_filter=1, stress=True, steps=16),
        # the middle of the range: graphite to diamond-like, 15 GPa
        _case("ts_4608_step", lattice="graphite", nx=12, ny=8, nz=6, images=24, steps=20,
              pressure=15.0),
        # the headline: the same at 98,304 atoms and 24 images, adaptive images
        _case("ts_98304_step", lattice="graphite", nx=32, ny=32, nz=12, images=24, steps=20, climb=100,
              refine=20, pressure=15.0),
        # the largest LJ band
        _case("lj_97555_step", nx=29, ny=29, nz=29, images=24, steps=20),
        # many bands of all sizes in one batch
        _case("batch_64_step", kind="batch", lattice="mix", nx=64, ny=256, nz=32000, images=17),
        # relaxing a band's endpoint
        _case("relax_lj_4000", kind="relax", nx=10, ny=10, nz=10, steps=64),
        # requests, one of each potential; candidate lists are built in each
        _case("request_lj_16383", kind="request", nx=16, ny=16, nz=16, images=11, steps=64),
        _case("request_ts_2743", kind="request", lattice="diamond", nx=7, ny=7, nz=7, images=13, steps=64),
        # the readout of a transition between the images
        _case("profile_ts_32832", kind="profile", lattice="graphite", nx=18, ny=19, nz=12, images=9, samples=257),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: any kind, lattice and precision, atom counts over
    their logarithm, at most the largest listed band's atoms x images x steps."""
    kind = rng.choice(["step", "step", "step", "step", "relax", "request", "profile", "batch"])
    if kind == "batch":
        return _case(kind=kind, lattice="mix", nx=rng.randint(9, 64), ny=rng.randint(200, 400),
                     nz=_log_int(rng, 2000, 32000), images=rng.randint(7, 17), steps=rng.randint(16, 40))
    fp64 = rng.random() < 0.25
    lattice = rng.choice(["fcc", "fcc", "diamond", "graphite"])
    if kind == "profile" and not fp64:  # slopes of FP32 hops are made of rounding, as above
        lattice = "graphite"
    atoms = _log_int(rng, 200, 97000 if kind == "step" else 30000)
    per = 4 if lattice == "fcc" else 8
    k = max(3.0 if lattice == "fcc" else 2.0, (atoms / per) ** (1.0 / 3.0))
    if lattice == "graphite":
        nz = 3 * max(1, int(round(k / 6)))  # 2 nz layers, a multiple of 6
        side = max(2.0, math.sqrt(atoms / (8.0 * nz)))
        nx, ny = max(2, int(side * rng.uniform(0.8, 1.25))), max(2, int(side * rng.uniform(0.8, 1.25)))
    else:
        lo = 3 if lattice == "fcc" else 2
        nx, ny, nz = (max(lo, int(round(k * rng.uniform(0.85, 1.15)))) for _ in range(3))
    hop = lattice != "graphite"
    images = rng.randint(5, 24) if atoms < 40000 else rng.randint(5, 20)
    return _case(kind=kind, lattice=lattice, nx=nx, ny=ny, nz=nz,
                 images=images, steps=rng.randint(10, 20) if kind == "step" else rng.randint(32, 64), fp64=fp64,
                 cell_filter=rng.choice([2, 2, 2, 1, 0]), pressure=0.0 if hop else rng.choice([0.0, 15.0]),
                 stress=rng.random() < 0.15, climb=50 if lattice == "fcc" and fp64 and atoms < 400 else -1,
                 refine=20 if lattice == "graphite" and kind == "step" and rng.random() < 0.5 else 0,
                 samples=rng.choice([0, 65, 257, 1023]) if kind == "profile" else 0)


# ------------------------------------------------------------------------ inputs
def _grid(nx, ny, nz, basis):
    g = np.stack(np.meshgrid(np.arange(nx), np.arange(ny), np.arange(nz), indexing="ij"), -1).reshape(-1, 1, 3)
    return (g + basis).reshape(-1, 3)


def _hop(lattice, nx, ny, nz):
    """Vacancy at site 0; in the final state its nearest neighbour has hopped into it."""
    a, basis, hop = (1.5496, FCC, 1) if lattice == "fcc" else (3.566, np.concatenate([FCC, FCC + 0.25]), 4)
    sites = _grid(nx, ny, nz, basis) * a
    pi = sites[1:].copy()
    pf = pi.copy()
    pf[hop - 1] = sites[0]
    h = np.diag([nx * a, ny * a, nz * a])
    return pi, h, pf, h.copy()


def _layers(nx, ny, layers, d, pitch, shift, pucker):
    s3 = math.sqrt(3.0)
    base = np.array([[0.0, 0.0], [0.0, d], [s3 * d / 2, 1.5 * d], [s3 * d / 2, 2.5 * d]])
    lat, ix, iy, b = np.meshgrid(np.arange(layers), np.arange(nx), np.arange(ny), np.arange(4), indexing="ij")
    pos = np.stack([base[b, 0] + ix * s3 * d, (base[b, 1] + iy * 3.0 * d + (lat % shift) * d) % (ny * 3.0 * d),
                    lat * pitch + np.array([-pucker, pucker, -pucker, pucker])[b]], -1).reshape(-1, 3)
    return pos, np.diag([nx * s3 * d, ny * 3.0 * d, layers * pitch])


def _graphite(nx, ny, nz):
    """AB graphite to the same atoms as a (111) stack of cubic diamond."""
    a = 3.566
    pi, hi = _layers(nx, ny, 2 * nz, 1.46, 3.35, 2, 0.0)
    pf, hf = _layers(nx, ny, 2 * nz, a / math.sqrt(6.0), a / math.sqrt(3.0), 3, a * math.sqrt(3.0) / 24.0)
    return pi, hi, pf, hf


def _endpoints(c, rng):
    pi, hi, pf, hf = _graphite(c["nx"], c["ny"], c["nz"]) if c["lattice"] == "graphite" else _hop(
        c["lattice"], c["nx"], c["ny"], c["nz"])
    if c["lattice"] == "graphite":
        pi, pf = (v + rng.normal(0.0, 0.01, v.shape) for v in (pi, pf))
    elif c["kind"] == "relax":
        pi = pi + rng.normal(0.0, 0.02, pi.shape)
    return pi, hi, pf, hf


def _noise(c, rng, atoms):
    """Zero-mean displacements of a hop's interior images, off the symmetric straight line."""
    if c["lattice"] == "graphite":
        return None
    d = rng.normal(0.0, 0.01, (c["images"] - 2, atoms, 3))
    return d - d.mean(axis=1, keepdims=True)


def _params(c):
    refine = c["refine"]
    p = cfneb.default_params(
        cfneb.CFNEB_LJ if c["lattice"] == "fcc" else cfneb.CFNEB_TERSOFF_C, force_fp64=1 if c["fp64"] else 0,
        n_images=c["images"], max_images=min(64, c["images"] + 16) if refine else c["images"], climb_after=c["climb"],
        cell_filter=c["cell_filter"], pressure_GPa=c["pressure"], refine_every=refine)
    if c["stress"]:
        for q in range(6):
            p.stress_GPa[q] = STRESS[q]
    return p


def _batch_members(c, seed):
    """nx bands, atom targets log-uniform in [ny, nz], 5 to `images` images, LJ and Tersoff in turn."""
    rng = np.random.default_rng([11, seed])
    out = []
    shape = np.random.default_rng([c["nx"], c["ny"], c["nz"]])  # the sizes are the case's, not the seed's
    for q in range(c["nx"]):
        atoms = math.exp(shape.uniform(math.log(c["ny"]), math.log(c["nz"])))
        lattice, per, lo = ("fcc", 4, 4) if q % 2 == 0 else ("diamond", 8, 2)
        k = max(lo, int(round((atoms / per) ** (1.0 / 3.0))))
        m = dict(DEFAULT, lattice=lattice, nx=k, ny=k, nz=max(lo, int(round(atoms / per / k / k))),
                 images=int(shape.integers(5, c["images"] + 1)))
        out.append((m, rng))
    return out


def _workspace(p, atoms):
    """Device memory for a band, and the coordinates of its image slots in it."""
    ws = torch.empty(cfneb.band_bytes(p, atoms) + 256, dtype=torch.uint8, device="cuda")
    at = -ws.data_ptr() % 256
    ld = (atoms + 3 + 63) // 64 * 64
    return ws, ws[at:at + p.max_images * 3 * ld * 8].view(torch.float64).view(p.max_images, 3, ld)


def prepare(case, seed):
    c = dict(DEFAULT, **case)
    if c["kind"] == "batch":
        batch, X = cfneb.Batch(c["nx"]), []
        for m, rng in _batch_members(c, seed):
            ends, p = _endpoints(m, rng), _params(m)
            ws, x = _workspace(p, len(ends[0]))
            slot = batch.add(p, *ends, workspace=ws)
            batch.bands[slot].displace_interior(_noise(m, rng, len(ends[0])))
            X.append(x)
        return dict(c=c, batch=batch, X=X)
    rng = np.random.default_rng([7, seed])
    ends, p = _endpoints(c, rng), _params(c)
    s = dict(c=c, p=p, ends=ends, noise=_noise(c, rng, len(ends[0])))
    if c["kind"] in ("step", "profile"):
        ws, s["X"] = _workspace(p, len(ends[0]))
        s["band"] = cfneb.Band(p, *ends, workspace=ws)
        if s["noise"] is not None:
            s["band"].displace_interior(s["noise"])
    return s


# -------------------------------------------------------------------------- pass
def _typed(c, v):
    return np.asarray(v, np.float64 if c["fp64"] else np.float32)


def _read(c, steps, fmax, e):
    out = dict(steps=int(steps), H=_typed(c, e["H"]), ci=int(e["ci"]))
    if c["fp64"] or c["lattice"] == "graphite":
        out.update(fmax=_typed(c, fmax), xi=_typed(c, e["xi"]))
    return out


def run(state):
    c = state["c"]
    if c["kind"] == "step":
        band = state["band"]
        steps, fmax, _ = band.step(c["steps"], 0.0)
        return dict(_read(c, steps, fmax, band.energies()), X=state["X"] if c["fp64"] else state["X"].float())
    if c["kind"] == "request":
        band = cfneb.Band(state["p"], *state["ends"])
        if state["noise"] is not None:
            band.displace_interior(state["noise"])
        steps, fmax, _ = band.step(c["steps"], 0.0)
        e = band.energies()
        pos, cell = band.get_image(len(e["H"]) // 2)
        band.close()
        return dict(_read(c, steps, fmax, e), pos=_typed(c, pos), cell=_typed(c, cell))
    if c["kind"] == "relax":
        pos, cell, steps, fmax, _ = cfneb.relax(state["p"], state["ends"][0], state["ends"][1], max_steps=c["steps"],
                                                f_tol=0.0)
        out = dict(steps=int(steps), pos=_typed(c, pos), cell=_typed(c, cell))
        return dict(out, fmax=_typed(c, fmax)) if c["fp64"] else out
    if c["kind"] == "profile":
        r = state["band"].profile(c["samples"])
        return dict(s=_typed(c, r["s"]), H=_typed(c, r["H"]), slope=_typed(c, r["slope"]),
                    samples=_typed(c, r["samples"]))
    batch = state["batch"]
    steps, conv, errs = batch.step(c["steps"], 0.0)
    es = [batch.energies(q) for q in range(c["nx"])]
    return dict(steps=steps, converged=conv.astype(np.int32), errors=errs,
                H=np.concatenate([_typed(c, e["H"]) for e in es]),
                X=torch.cat([x.reshape(-1).float() for x in state["X"]]))


def _atoms(c):
    if c["lattice"] == "graphite":
        return 8 * c["nx"] * c["ny"] * c["nz"]
    return (4 if c["lattice"] == "fcc" else 8) * c["nx"] * c["ny"] * c["nz"] - 1


def _step_work(c, images):
    """Per band step: coordinates and velocities of every moving row read and written once;
    11 operations per neighbour within rc (78 of them in the LJ crystal; each pair once) or
    about 790 per carbon atom, and about 150 for projection, filter and optimizer."""
    rows = (_atoms(c) + 3) * images
    return 96.0 * rows, (150.0 + (11 * 78 if c["lattice"] == "fcc" else 790)) * rows


def work(case):
    c = dict(DEFAULT, **case)
    if c["kind"] == "batch":
        members = [m for m, _ in _batch_members(c, 0)]
        parts = [_step_work(m, m["images"] - 2) for m in members]
        return dict(bytes=c["steps"] * sum(p[0] for p in parts), flops=c["steps"] * sum(p[1] for p in parts))
    ends = 48.0 * _atoms(c)
    if c["kind"] == "profile":
        b, f = _step_work(c, c["images"])
        return dict(bytes=b / 4, flops=f)
    if c["kind"] == "relax":
        b, f = _step_work(c, 1)
        return dict(bytes=b * c["steps"] + 2 * ends, flops=f * (c["steps"] + 1))
    b, f = _step_work(c, c["images"] - 2)
    if c["kind"] == "request":
        return dict(bytes=b * c["steps"] + 2 * ends, flops=f * (c["steps"] + 1))
    return dict(bytes=b * c["steps"], flops=f * c["steps"])


# ------------------------------------------------- the same in 64 bits, plain torch
DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _neighbours(R, h, rc):
    """Every (i, j, d) with d = R_j + n h - R_i, 0 < |d| < rc, by a linked-cell search."""
    hi = torch.linalg.inv(h)
    s = R @ hi
    fl = torch.floor(s)
    s = s - fl
    Rw = s @ h
    w = 1.0 / torch.linalg.norm(hi, dim=0)
    n = len(R)
    nb = [max(1, min(int(float(w[q]) / (rc * (1 + 1e-9))), int(n ** (1 / 3)) + 1)) for q in range(3)]
    reach = [max(1, math.ceil(rc / (float(w[q]) / nb[q]))) for q in range(3)]
    b = [(s[:, q] * nb[q]).long().clamp(0, nb[q] - 1) for q in range(3)]
    key = (b[0] * nb[1] + b[1]) * nb[2] + b[2]
    order = torch.argsort(key, stable=True)
    count = torch.bincount(key, minlength=nb[0] * nb[1] * nb[2])
    start = torch.cumsum(count, 0) - count
    me = torch.arange(n, device=R.device)
    found = []
    for o0 in range(-reach[0], reach[0] + 1):
        for o1 in range(-reach[1], reach[1] + 1):
            for o2 in range(-reach[2], reach[2] + 1):
                t = [b[0] + o0, b[1] + o1, b[2] + o2]
                m = [torch.div(t[q], nb[q], rounding_mode="floor") for q in range(3)]
                kb = ((t[0] - m[0] * nb[0]) * nb[1] + (t[1] - m[1] * nb[1])) * nb[2] + (t[2] - m[2] * nb[2])
                k = count[kb]
                i = torch.repeat_interleave(me, k)
                local = torch.arange(len(i), device=R.device) - (torch.cumsum(k, 0) - k)[i]
                j = order[start[kb][i] + local]
                d = Rw[j] - Rw[i] + (torch.stack(m, -1).double() @ h)[i]
                r2 = (d * d).sum(1)
                ok = (r2 < rc * rc) & (r2 > 1e-12)
                found.append((i[ok], j[ok], d[ok]))
    return tuple(torch.cat([f[q] for f in found]) for q in range(3))


def _lj(p, R, h):
    i, j, d = _neighbours(R, h, p.lj_rc)
    r2 = (d * d).sum(1)
    s6 = (p.lj_sigma ** 2 / r2) ** 3
    c6 = (p.lj_sigma ** 2 / p.lj_rc ** 2) ** 3
    E = 0.5 * (4 * p.lj_eps * (s6 * s6 - s6) - (4 * p.lj_eps * (c6 * c6 - c6) if p.lj_shift else 0.0)).sum()
    f = (24 * p.lj_eps * (s6 - 2 * s6 * s6) / r2)[:, None] * d
    return E, torch.zeros_like(R).index_add_(0, i, f), -0.5 * _outer_sum(d, f)


def _outer_sum(a, b):
    return torch.stack([(a[:, q:q + 1] * b).sum(0) for q in range(3)])


def _tersoff(p, R, h):
    i, j, d = _neighbours(R, h, p.ts_S)
    order = torch.argsort(i, stable=True)
    i, j, d = i[order], j[order], d[order].detach().requires_grad_(True)
    n = len(R)
    k = torch.bincount(i, minlength=n)
    B = int(k.max()) if len(i) else 1
    at = torch.arange(len(i), device=R.device) - (torch.cumsum(k, 0) - k)[i]
    pad = torch.zeros(n, B, 3, dtype=R.dtype, device=R.device)
    pad[..., 0] = 10 * p.ts_S  # no bond: beyond the cutoff
    with torch.enable_grad():
        v = pad.index_put((i, at), d)
        r = v.square().sum(-1).sqrt()
        fc = torch.where(r < p.ts_R, torch.ones_like(r), torch.where(
            r < p.ts_S, 0.5 + 0.5 * torch.cos(math.pi * (r - p.ts_R) / (p.ts_S - p.ts_R)), torch.zeros_like(r)))
        u = v / r[..., None]
        cos = (u[:, :, None] * u[:, None]).sum(-1)
        x = (p.ts_h - cos) ** 2
        g = 1 + (p.ts_c ** 2 / p.ts_d ** 2) * x / (p.ts_d ** 2 + x)
        other = 1.0 - torch.eye(B, dtype=R.dtype, device=R.device)
        zeta = (fc[:, None] * g * other).sum(-1)
        bz = torch.where(zeta > 0, p.ts_beta * zeta, torch.full_like(zeta, 1e-300))
        bo = (1 + bz ** p.ts_n) ** (-0.5 / p.ts_n)
        E = 0.5 * (fc * (p.ts_A * torch.exp(-p.ts_lambda1 * r) - bo * p.ts_B * torch.exp(-p.ts_lambda2 * r))).sum()
        (P,) = torch.autograd.grad(E, d)
    d = d.detach()
    F = torch.zeros_like(R).index_add_(0, i, P).index_add_(0, j, -P)
    return E.detach(), F, -_outer_sum(d, P)


class _Exact:
    """One band (or, with `relax`, one structure) in 64 bits."""

    def __init__(self, p, ends, relax=False):
        t = lambda v: torch.tensor(v, dtype=torch.float64, device=DEV)  # noqa: E731
        pi, hi, pf, hf = (t(v) for v in ends)
        self.p, self.h0, self.relax = p, hi, relax
        n = self.n = len(pi)
        det = abs(float(torch.linalg.det(hi)))
        self.omega0 = det
        self.cf = p.cell_factor if p.cell_factor > 0 else det ** (1 / 3) * n ** (1 / 6)
        h0i = torch.linalg.inv(hi)
        ds = pf @ torch.linalg.inv(hf) - pi @ h0i
        ds = ds - torch.round(ds)
        D = h0i @ hf
        eye = torch.eye(3, dtype=torch.float64, device=DEV)
        a = torch.cat([pi, self.cf * eye])
        b = torch.cat([pi + ds @ hi, self.cf * (D if p.cell_filter == 1 else D @ D.T)])
        M = 3 if relax else p.n_images
        self.X = [a + (k / (M - 1)) * (b - a) if 0 < k < M - 1 else (a.clone() if k == 0 else b.clone())
                  for k in range(M)]
        self.V = [torch.zeros_like(a) for _ in range(M)]
        v = p.stress_GPa
        self.S = t([[v[0], v[5], v[4]], [v[5], v[1], v[3]], [v[4], v[3], v[2]]]) / GPA
        self.ev = [self.evaluate(x) for x in self.X]
        self.H = [e[0] for e in self.ev]
        self.dt, self.alpha, self.npos, self.fresh, self.step_no, self.ci = p.fire_dt0, p.fire_astart, 0, True, 0, -1
        self.fmax = 0.0

    def deform(self, X):
        B = X[self.n:] / self.cf
        if self.p.cell_filter == 1:
            return B
        w, q = torch.linalg.eigh(0.5 * (B + B.T))
        return q @ torch.diag(torch.sqrt(w)) @ q.T

    def evaluate(self, X):
        """(enthalpy, generalized force) of one image."""
        p, n = self.p, self.n
        D = self.deform(X)
        h = self.h0 @ D
        E, F, V = (_lj if p.potential == cfneb.CFNEB_LJ else _tersoff)(p, X[:n] @ D, h)
        om = torch.abs(torch.linalg.det(h))
        eye = torch.eye(3, dtype=torch.float64, device=DEV)
        press = p.pressure_GPa / GPA
        H = E + press * om - self.omega0 * (self.S * (0.5 * (D @ D.T - eye))).sum()
        Ve = V - press * om * eye + self.omega0 * D.T @ self.S @ D
        Di = torch.linalg.inv(D)
        G = Di.T @ Ve
        if p.cell_filter == 1:
            G = G / self.cf
        else:
            G = G @ Di
            G = 0.5 * (G + G.T) * (p.b_force_scale / self.cf if p.cell_filter == 2 else 0.0)
        return float(H), torch.cat([F @ D.T, G])

    def centred(self, v):
        v = v.clone()
        v[:self.n] -= v[:self.n].mean(0)
        return v

    @staticmethod
    def weights(Hm, H0, Hp):
        if Hp > H0 > Hm:
            return 1.0, 0.0
        if Hp < H0 < Hm:
            return 0.0, 1.0
        big, small = max(abs(Hp - H0), abs(Hm - H0)), min(abs(Hp - H0), abs(Hm - H0))
        return (big, small) if Hp > Hm else (small, big)

    def step(self):
        p, X = self.p, self.X
        M = len(X)
        for k in range(1, M - 1):
            self.H[k], F = self.evaluate(X[k])
            self.ev[k] = (self.H[k], F)
        self.ci = -1
        if not self.relax and p.climb_after >= 0 and self.step_no >= p.climb_after:
            self.ci = max(range(1, M - 1), key=lambda k: (self.H[k], -k))
        fn = [None] * M
        for k in range(1, M - 1):
            F = self.centred(self.ev[k][1])
            fn[k] = F
            if self.relax:
                continue
            tp, tm = self.centred(X[k + 1] - X[k]), self.centred(X[k] - X[k - 1])
            a, b = self.weights(self.H[k - 1], self.H[k], self.H[k + 1])
            tau = a * tp + b * tm
            norm = float(tau.norm())
            if norm > 0:
                tau = tau / norm
                ft = (F * tau).sum()
                fn[k] = F + tau * (-2 * ft if k == self.ci else p.k_spring * (tp.norm() - tm.norm()) - ft)
        cv, cf, dt, alpha, npos = 1.0, 0.0, self.dt, self.alpha, self.npos
        inner = range(1, M - 1)
        if not self.fresh:
            P = sum(float((fn[k] * self.V[k]).sum()) for k in inner)
            if P > 0:
                FF = math.sqrt(sum(float((fn[k] ** 2).sum()) for k in inner))
                VV = math.sqrt(sum(float((self.V[k] ** 2).sum()) for k in inner))
                if FF > 0:
                    cv, cf = 1 - alpha, alpha * VV / FF
                if npos > p.fire_nmin:
                    dt, alpha = min(dt * p.fire_finc, p.fire_dtmax), alpha * p.fire_fa
                npos += 1
            else:
                cv, cf, alpha, dt, npos = 0.0, 0.0, p.fire_astart, dt * p.fire_fdec, 0
        self.fmax = max(float(fn[k].norm(dim=1).max()) for k in inner)
        V = [None if fn[k] is None else cv * self.V[k] + cf * fn[k] + dt * fn[k] for k in range(M)]
        big = max(float((dt * V[k]).norm(dim=1).max()) for k in inner)
        scale = p.fire_maxstep / big if big > p.fire_maxstep else 1.0
        for k in inner:
            self.V[k] = V[k]
            X[k] = X[k] + scale * dt * V[k]
        self.dt, self.alpha, self.npos, self.fresh = dt, alpha, npos, False
        self.step_no += 1
        if not self.relax and p.refine_every > 0 and self.step_no % p.refine_every == 0:
            self.refine()

    def refine(self):
        p, X = self.p, self.X
        M = len(X)
        d2 = [float((X[k + 1] - X[k]).square().sum()) for k in range(M - 1)]
        total, k = sum(d2), max(range(M - 1), key=lambda q: (d2[q], -q))
        if M < p.max_images and p.ins_den * (M - 1) * d2[k] > p.ins_num * total:
            X.insert(k + 1, X[k] + 0.5 * (X[k + 1] - X[k]))
            self.H.insert(k + 1, 0.5 * (self.H[k] + self.H[k + 1]))
            self.ev.insert(k + 1, None)
        else:
            inner = [q for q in range(1, M - 1) if q != self.ci]
            if M <= p.min_images or not inner:
                return
            j = min(inner, key=lambda q: (max(d2[q - 1], d2[q]), q))
            if not p.del_den * (M - 1) * max(d2[j - 1], d2[j]) < p.del_num * total:
                return
            del X[j], self.H[j], self.ev[j]
        self.V = [torch.zeros_like(x) for x in X]
        self.alpha, self.npos, self.fresh, self.ci = p.fire_astart, 0, True, -1

    def arc(self):
        s = [0.0]
        for k in range(len(self.X) - 1):
            s.append(s[-1] + float(self.centred(self.X[k + 1] - self.X[k]).norm()))
        return np.array(s)

    def image(self, k):
        D = self.deform(self.X[k])
        return (self.X[k][:self.n] @ D).cpu().numpy(), (self.h0 @ D).cpu().numpy()

    def profile(self, samples):
        M, X = len(self.X), self.X
        s, H, slope = self.arc(), np.array(self.H), np.zeros(len(self.X))
        for k in range(M):
            tp = self.centred(X[k + 1] - X[k]) if k < M - 1 else None
            tm = self.centred(X[k] - X[k - 1]) if k > 0 else None
            a, b = (1.0, 0.0) if k == 0 else (0.0, 1.0) if k == M - 1 else self.weights(H[k - 1], H[k], H[k + 1])
            tau = sum(w * v for w, v in ((a, tp), (b, tm)) if v is not None)
            if float(tau.norm()) > 0:
                slope[k] = -float((self.centred(self.ev[k][1]) * tau).sum() / tau.norm())
        x = np.arange(samples) / max(1, samples - 1) * s[-1]
        k = np.clip(np.searchsorted(s, x, side="right") - 1, 0, M - 2)
        d = s[k + 1] - s[k]
        t = (x - s[k]) / d
        y = ((1 + 2 * t) * (1 - t) ** 2 * H[k] + t * (1 - t) ** 2 * d * slope[k] + t * t * (3 - 2 * t) * H[k + 1]
             - t * t * (1 - t) * d * slope[k + 1])
        return s, H, slope, y


def exact(case, seed):
    c = dict(DEFAULT, **case)
    rng = np.random.default_rng([7, seed])
    images = {"relax": 1, "batch": 1000}.get(c["kind"], c["images"])
    steps = 1 if c["kind"] == "profile" else c["steps"]
    # about 3 ms an image and step, and 40 ns an atom of carbon or 250 ns of LJ
    if c["kind"] == "batch" or images * steps * (3e-3 + _atoms(c) * (2.5e-7 if c["lattice"] == "fcc" else 4e-8)) > 16.0:
        return None
    ends, p = _endpoints(c, rng), _params(c)
    noise = _noise(c, rng, len(ends[0]))
    if c["kind"] == "relax":
        ends = (ends[0], ends[1], ends[0], ends[1])
    b = _Exact(p, ends, relax=c["kind"] == "relax")
    if noise is not None and c["kind"] != "relax":
        for k in range(1, c["images"] - 1):
            b.X[k][:b.n] += torch.tensor(noise[k - 1], device=DEV)
            b.H[k], F = b.evaluate(b.X[k])
            b.ev[k] = (b.H[k], F)
    if c["kind"] == "profile":
        s, H, slope, y = b.profile(c["samples"])
        return dict(s=s, H=H, slope=slope, samples=y)
    for _ in range(c["steps"]):
        b.step()
    if c["kind"] == "relax":
        pos, cell = b.image(1)
        return dict(steps=c["steps"], fmax=np.asarray(b.fmax), pos=pos, cell=cell)
    s = b.arc()
    out = dict(steps=c["steps"], fmax=np.asarray(b.fmax), H=np.array(b.H), xi=s / s[-1], ci=b.ci)
    if c["kind"] == "request":
        out["pos"], out["cell"] = b.image(len(b.X) // 2)
        return out
    X = torch.zeros(p.max_images, 3, (b.n + 3 + 63) // 64 * 64, dtype=torch.float64)
    for k, x in enumerate(b.X):  # an image inserted on the way has the first free slot
        X[k, :, :b.n + 3] = x.T.cpu()
    return dict(out, X=X if len(b.X) == c["images"] else None)
