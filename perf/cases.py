"""The measured cases: what a program that uses this library has it do.

Every case is one call (or the few calls of one step) through the package's
public entry points, on inputs made from a seed on the GPU.  ``op`` names the
path:

* ``substeps``  acoustic_substeps, a few substeps of a time loop;
* ``tracers``   tracer_transport with the fluxes a run has accumulated;
* ``dynamics``  one pass of the remapping loop (substeps, tracers, remap);
* ``ensemble``  many uneven members at once, replayed from a HIP graph;
* ``sums``      the conservation diagnostics of a step;
* ``train``     minibatches of the learned correction's network;
* ``correct``   features, network and correction applied to a coarse state.

States evolve from pass to pass, as in a time loop.  The cube states are the
analytic baroclinic jet (balanced zonal jet in discretely hydrostatic columns
on evenly spaced sigma layers) with N(0, 1) m/s noise on the winds, the doubly
periodic ones an isothermal 300 K column with a mean wind of 10 m/s and noise.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2205_04148_amd as fv3

H = 3
GRAV, RDGAS, CP_AIR, P0 = 9.80665, 287.05, 1004.6, 1.0e5
KAPPA = RDGAS / CP_AIR
RADIUS, OMEGA, PTOP = fv3.RADIUS, fv3.OMEGA, 100.0

# The options a run turns on beside the plain scheme: damping, off-centring,
# the unlimited order, cubic interface pressure and humidity ("physics"), and
# the tile-edge treatments of the cube ("edges").
OPTIONS = {
    "plain": {},
    "physics": dict(beta=0.75, hord=6, pp_order=4, nord=1, d4_bg=0.12, d2_bg=0.02, dddmp=0.1, vtdm=0.03),
    "edges": dict(edge_fix=True, edge_ppm=True, edge_interp=True),
}

PROGNOSTIC = ("u", "v", "w", "delp", "pt", "delz")
DIAGNOSTIC = ("uc", "vc", "mfx", "mfy", "cx", "cy", "dp0", "pfull", "phi")


def listed():
    return [
        # the smallest configuration of the tests and the smoke check: one
        # plane of 48 x 48 points per layer, bound by launches
        dict(name="periodic_48x8_fp64", op="substeps", kind=0, n=48, nz=8, precision="fp64", n_split=10,
             options="plain"),
        # the middle cubed-sphere resolution, in the reference precision
        dict(name="cube_96x79_fp64", op="substeps", kind=1, n=96, nz=79, precision="fp64", n_split=2,
             options="plain"),
        # the benchmark's resolution, in both precisions
        dict(name="cube_192x79_mixed", op="substeps", kind=1, n=192, nz=79, precision="mixed", n_split=2,
             options="plain"),
        dict(name="cube_192x79_fp64", op="substeps", kind=1, n=192, nz=79, precision="fp64", n_split=2,
             options="plain"),
        # a run with humidity and every damping option, on sizes that divide
        # by none of the block sizes
        dict(name="cube_77x37_physics_mixed", op="substeps", kind=1, n=77, nz=37, precision="mixed", n_split=2,
             options="physics"),
        # a run with the tile-edge treatments
        dict(name="cube_49x33_edges_fp64", op="substeps", kind=1, n=49, nz=33, precision="fp64", n_split=2,
             options="edges"),
        # the tracer transport of the benchmark step (two sub-cycles)
        dict(name="tracers_192x79_mixed", op="tracers", kind=1, n=192, nz=79, precision="mixed", nq=4, hord_tr=0),
        # the coarse model of the learned correction in its remapping loop
        dict(name="dynamics_48x79_mixed", op="dynamics", kind=1, n=48, nz=79, precision="mixed", nq=4, k_split=2,
             n_split=3),
        # serving many small independent runs on one GPU
        dict(name="ensemble_8_mixed", op="ensemble", members=8, n_lo=64, n_hi=160, nz_lo=32, nz_hi=79,
             precision="mixed", n_split=2),
        # the mass diagnostics of the benchmark step
        dict(name="sums_192x79_mixed", op="sums", kind=1, n=192, nz=79, precision="mixed", nq=4),
        # training and using the learned correction at its own sizes
        dict(name="train_4096x79", op="train", rows=4096, nz=79, hidden=256, batches=4),
        dict(name="correct_48x79_mixed", op="correct", kind=1, n=48, nz=79, precision="mixed", hidden=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["substeps"] * 6 + ["tracers", "dynamics", "ensemble", "sums", "train", "correct"])
    precision = rng.choice(["fp64", "mixed"])
    kind = rng.choice([0, 1, 1])
    n, nz = _log_int(rng, 20, 188), _log_int(rng, 5, 79)
    if op == "substeps":
        options = rng.choice(["plain", "plain", "physics", "edges"] if kind else ["plain", "plain", "physics"])
        return dict(op=op, kind=kind, n=n, nz=nz, precision=precision, n_split=rng.randint(1, 2), options=options)
    if op == "tracers":
        return dict(op=op, kind=kind, n=n, nz=nz, precision=precision, nq=rng.randint(1, 7),
                    hord_tr=rng.choice([0, 0, 5, 6, 7]))
    if op == "dynamics":
        return dict(op=op, kind=kind, n=_log_int(rng, 20, 96), nz=nz, precision=precision, nq=rng.randint(0, 5),
                    k_split=rng.randint(1, 2), n_split=rng.randint(1, 3))
    if op == "ensemble":
        n_lo, nz_lo = _log_int(rng, 16, 64), rng.randint(5, 32)
        return dict(op=op, members=rng.randint(2, 8), n_lo=n_lo, n_hi=n_lo + rng.randint(5, 90), nz_lo=nz_lo,
                    nz_hi=nz_lo + rng.randint(1, 40), precision=precision, n_split=rng.randint(1, 2))
    if op == "sums":
        return dict(op=op, kind=kind, n=n, nz=nz, precision=precision, nq=rng.randint(0, 6))
    if op == "train":
        return dict(op=op, rows=_log_int(rng, 200, 4096), nz=_log_int(rng, 8, 79), hidden=16 * rng.randint(2, 16),
                    batches=rng.randint(1, 4))
    return dict(op=op, kind=1, n=_log_int(rng, 12, 60), nz=_log_int(rng, 8, 79), precision=precision,
                hidden=16 * rng.randint(2, 16))


# ------------------------------------------------------------------ inputs
# Grids depend on no input and are shared by all states of a program: the
# latest few are kept.
_GRIDS: dict = {}


def _grid(kind, n, nz, precision, **options):
    key = (kind, n, nz, precision, tuple(sorted(options.items())))
    if key not in _GRIDS:
        while len(_GRIDS) >= 10:
            del _GRIDS[next(iter(_GRIDS))]
        _GRIDS[key] = fv3.Grid(kind, n, nz, ptop=PTOP, precision=precision, **options)
    return _GRIDS[key]


def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, dtype=torch.float64, device="cuda")


def _uniform(gen, *shape):
    return torch.rand(shape, generator=gen, dtype=torch.float64, device="cuda")


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True)


FRAMES = (((1, 0, 0), (0, 1, 0), (0, 0, 1)), ((0, 1, 0), (-1, 0, 0), (0, 0, 1)), ((0, 0, 1), (-1, 0, 0), (0, -1, 0)),
          ((-1, 0, 0), (0, -1, 0), (0, 0, 1)), ((0, -1, 0), (1, 0, 0), (0, 0, 1)), ((0, 0, -1), (0, 1, 0), (1, 0, 0)))


def _corners(n):
    """Lattice corners of the six equiangular gnomonic tiles, [6][n+1][n+1][3]."""
    f = torch.tensor(FRAMES, dtype=torch.float64, device="cuda")
    a = torch.tan((2 * torch.arange(n + 1, dtype=torch.float64, device="cuda") - n) * (math.pi / (4 * n)))
    return _unit(f[:, 0, None, None] + a[None, None, :, None] * f[:, 1, None, None] +
                 a[None, :, None, None] * f[:, 2, None, None])


class Jet:
    """Balanced baroclinic jet in closed form (temperature, pressure and zonal
    wind of latitude and height)."""

    te, tp, lapse, b, K = 310.0, 240.0, 0.005, 2.0, 3
    t0 = 0.5 * (te + tp)
    B = (t0 - tp) / (t0 * tp)
    C = 0.5 * (K + 2) * (te - tp) / (te * tp)

    def __init__(self, lat):
        c = torch.cos(lat)
        self.c = c
        self.F = c ** self.K - self.K / (self.K + 2.0) * c ** (self.K + 2)
        self.G = self.K * (c ** (self.K - 1) - c ** (self.K + 1))

    def profile(self, z):
        zeta = z / (self.b * RDGAS * self.t0 / GRAV)
        e, ez = torch.exp(-zeta * zeta), torch.exp(self.lapse * z / self.t0)
        tau1 = ez / self.t0 + self.B * (1 - 2 * zeta * zeta) * e
        tau2 = self.C * (1 - 2 * zeta * zeta) * e
        temp = 1 / (tau1 - tau2 * self.F)
        logp = -(GRAV / RDGAS) * ((ez - 1) / self.lapse + self.B * z * e) + (GRAV / RDGAS) * self.C * z * e * self.F
        return temp, logp, self.C * z * e

    def height(self, p):
        """Height at pressure p, by Newton steps on log p."""
        z = -(RDGAS * self.t0 / GRAV) * torch.full_like(self.F, math.log(p / P0))
        for _ in range(12):
            temp, logp, _ = self.profile(z)
            z = z + (logp - math.log(p / P0)) * RDGAS * temp / GRAV
        return z

    def wind(self, z):
        temp, _, itau2 = self.profile(z)
        rc = RADIUS * self.c
        return -OMEGA * rc + torch.sqrt((OMEGA * rc) ** 2 + rc * (GRAV / RADIUS) * itau2 * self.G * temp)


def _layers(nz):
    pi = [PTOP + (P0 - PTOP) * k / nz for k in range(nz + 1)]
    bar = [(pi[k + 1] - pi[k]) / math.log(pi[k + 1] / pi[k]) for k in range(nz)]
    return pi, bar


def _put(g, buf, levels, x):
    nj, ni = x.shape[-2:]
    g.view(buf, levels)[:, :, H:H + nj, H:H + ni].copy_(x)


def _fill_state(g, s, seed):
    """Initial values of the grid's kind into state s; returns the generator."""
    gen, n, nz, f = _rng(seed), g.n, g.nz, s.f
    pi, bar = _layers(nz)
    if g.kind == 0:
        for k, sl in (("u", (n + 1, n)), ("v", (n, n + 1))):
            x = torch.empty(1, nz, *sl, dtype=torch.float64, device="cuda")
            x[:, :, :n, :n] = 10.0 + _normal(gen, 1, nz, n, n)
            if k == "u":
                x[:, :, n] = x[:, :, 0]
            else:
                x[:, :, :, n] = x[:, :, :, 0]
            _put(g, f[k], nz, x)
        temp = 300.0 + 0.1 * _normal(gen, 1, nz, n, n)
        for k in range(nz):
            lnr, sl = math.log(pi[k + 1] / pi[k]), (slice(None), k, slice(H, H + n), slice(H, H + n))
            g.view(f["delp"], nz)[sl] = pi[k + 1] - pi[k]
            g.view(f["pt"], nz)[sl] = (temp[:, k] * (P0 / bar[k]) ** KAPPA).to(f["pt"].dtype)
            g.view(f["delz"], nz)[sl] = -(RDGAS * temp[:, k] / GRAV) * lnr
        return gen
    B = _corners(n)
    lat = torch.asin(_unit(B[:, :-1, :-1] + B[:, 1:, :-1] + B[:, 1:, 1:] + B[:, :-1, 1:])[..., 2])
    jet = Jet(lat)
    z0, sl = None, (slice(H, H + n), slice(H, H + n))
    for k in range(nz + 1):
        z1 = jet.height(pi[k]) if k < nz else torch.zeros_like(lat)
        if k:
            lnr = math.log(pi[k] / pi[k - 1])
            temp = -GRAV * (z1 - z0) / (RDGAS * lnr)
            g.view(f["delp"], nz)[:, k - 1][:, sl[0], sl[1]] = pi[k] - pi[k - 1]
            g.view(f["pt"], nz)[:, k - 1][:, sl[0], sl[1]] = (temp * (P0 / bar[k - 1]) ** KAPPA).to(f["pt"].dtype)
            g.view(f["delz"], nz)[:, k - 1][:, sl[0], sl[1]] = z1 - z0
        z0 = z1
    for name, a, b in (("u", B[:, :, :-1], B[:, :, 1:]), ("v", B[:, :-1], B[:, 1:])):
        mid, d = _unit(a + b), b - a
        tan = _unit(d - (d * mid).sum(-1, keepdim=True) * mid)
        east = _unit(torch.stack([-mid[..., 1], mid[..., 0], torch.zeros_like(mid[..., 0])], -1))
        proj, face = (east * tan).sum(-1), Jet(torch.asin(mid[..., 2]))
        out = g.view(f[name], nz)
        nj, ni = proj.shape[-2:]
        for k in range(nz):
            x = face.wind(face.height(bar[k])) * proj + _normal(gen, 6, nj, ni)
            out[:, k, H:H + nj, H:H + ni] = x.to(out.dtype)
    return gen


def _bdt(kind, n):
    """Substep length: 15 s at C192 (Courant number kept), 0.2 s at 1 km spacing."""
    return 2880.0 / n if kind == 1 else 0.2


def _views(g, s, names):
    """Interior of the named fields, as views of the state's own buffers."""
    n, out = g.n, {}
    for k in names:
        L = g.nz + 1 if k in ("pfull", "phi") else g.nz
        ni, nj = n + (k in ("v", "uc", "mfx", "cx")), n + (k in ("u", "vc", "mfy", "cy"))
        out[k] = g.view(s.f[k], L)[:, :, H:H + nj, H:H + ni]
    return out


def _state(g, seed):
    s = fv3.State.allocate(g)
    return s, _fill_state(g, s, seed)


def _tracers(g, gen, nq):
    qs = []
    for _ in range(nq):
        q = g.new_field(g.nz)
        for k in range(g.nz):
            g.view(q, g.nz)[:, k, H:H + g.n, H:H + g.n] = _uniform(gen, g.T, g.n, g.n).to(q.dtype)
        qs.append(q)
    return qs


def _interior(g, q):
    return g.view(q, g.nz)[:, :, H:H + g.n, H:H + g.n]


def _hybrid(nz):
    """Reference interfaces ak + bk ps: pressure above, sigma towards the surface."""
    eta = np.arange(nz + 1) / nz
    bk = np.clip((eta - 0.3) / 0.7, 0.0, None) ** 2
    ak = PTOP + (P0 - PTOP) * eta - bk * P0
    ak[0], bk[0], ak[-1], bk[-1] = PTOP, 0.0, 0.0, 1.0
    return ak, bk


def _net_params(case, seed):
    sizes = (5 * case["nz"], case["hidden"], case["hidden"], 3 * case["nz"])
    r, out = np.random.default_rng(int(seed)), []
    for a, b in zip(sizes[:-1], sizes[1:]):
        out += [(r.standard_normal((a, b)) / math.sqrt(a)).astype(np.float32), np.zeros(b, np.float32)]
    return out


def _batches(case, seed):
    """Standardised columns and targets that depend on them."""
    gen, nz, out = _rng(seed), case["nz"], []
    mix = _normal(gen, 5 * nz, 3 * nz) / math.sqrt(5 * nz)
    for _ in range(case["batches"]):
        X = _normal(gen, case["rows"], 5 * nz)
        T = torch.tanh(X @ mix) + 0.1 * _normal(gen, case["rows"], 3 * nz)
        out.append((X.float(), T.float()))
    return out


def prepare(case, seed):
    op = case["op"]
    if op == "substeps":
        g = _grid(case["kind"], case["n"], case["nz"], case["precision"], **OPTIONS[case["options"]])
        s, gen = _state(g, seed)
        if case["options"] == "physics":
            s.f["qv"] = g.new_field(g.nz)
            _put(g, s.f["qv"], g.nz, 0.015 * _uniform(gen, g.T, g.nz, g.n, g.n))
        return dict(case, g=g, s=s, dt=case["n_split"] * _bdt(g.kind, g.n), out=_views(g, s, PROGNOSTIC + DIAGNOSTIC))
    if op == "tracers":
        # the fluxes of one substep, scaled to the hundred of a remapping step
        g = _grid(case["kind"], case["n"], case["nz"], case["precision"], hord_tr=case["hord_tr"])
        s, gen = _state(g, seed)
        fv3.acoustic_substeps(s, g, _bdt(g.kind, g.n), 1)
        for k in ("mfx", "mfy", "cx", "cy"):
            s.f[k] *= 100.0
        qs = _tracers(g, gen, case["nq"])
        return dict(case, g=g, s=s, qs=qs, out=[_interior(g, q) for q in qs])
    if op == "dynamics":
        g = _grid(case["kind"], case["n"], case["nz"], case["precision"])
        s, gen = _state(g, seed)
        qs = _tracers(g, gen, case["nq"])
        ak, bk = _hybrid(g.nz)
        out = _views(g, s, PROGNOSTIC)
        out["q"] = [_interior(g, q) for q in qs]
        return dict(case, g=g, s=s, qs=qs, ak=ak, bk=bk, out=out,
                    dt=case["k_split"] * case["n_split"] * _bdt(g.kind, g.n))
    if op == "ensemble":
        sizes, m = np.random.default_rng(4), case["members"]
        ns = sizes.integers(case["n_lo"], case["n_hi"] + 1, m)
        nzs = sizes.integers(case["nz_lo"], case["nz_hi"] + 1, m)
        gs = [_grid(0, int(a), int(b), case["precision"]) for a, b in zip(ns, nzs)]
        ss = [_state(g, 1000 * seed + k)[0] for k, g in enumerate(gs)]
        ens = fv3.Ensemble(ss, gs, case["n_split"] * _bdt(0, 0), case["n_split"], graph=True)
        return dict(case, ens=ens, out=[_views(g, s, PROGNOSTIC) for g, s in zip(gs, ss)])
    if op == "sums":
        g = _grid(case["kind"], case["n"], case["nz"], case["precision"])
        s, gen = _state(g, seed)
        # layer thicknesses of a run under way
        g.view(s.f["delp"], g.nz)[:, :, H:H + g.n, H:H + g.n] *= (
            1 + 0.01 * _normal(gen, g.T, g.nz, g.n, g.n)).to(s.f["delp"].dtype)
        return dict(case, g=g, s=s, qs=_tracers(g, gen, case["nq"]))
    if op == "train":
        net = fv3.MLP(_net_params(case, seed), maxrows=case["rows"])
        return dict(case, net=net, batches=_batches(case, seed))
    # correct: a coarse state, statistics of its own columns, a network of trained size
    g = _grid(case["kind"], case["n"], case["nz"], case["precision"])
    s, gen = _state(g, seed)
    rows, F = g.T * g.n * g.n, 5 * g.nz
    X, Y = torch.zeros(rows, F, device="cuda"), torch.zeros(rows, 3 * g.nz, device="cuda")
    zero, one = torch.zeros(F, device="cuda"), torch.ones(F, device="cuda")
    fv3.column_features(s, g, zero, one, X)
    mean, inv = X.mean(0), 1.0 / (X.std(0) + 1e-2)
    Z = (X - mean) * inv
    lo, hi = Z.amin(0).contiguous(), Z.amax(0).contiguous()
    ymean = 1e-7 * _normal(gen, 3 * g.nz).float()
    ystd = (1e-7 * (1 + _uniform(gen, 3 * g.nz))).float()
    net = fv3.MLP(_net_params(case, seed), maxrows=rows)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = dict(_views(g, s, ("u", "v", "pt")), X=X, Y=Y, flag=flag)
    return dict(case, g=g, s=s, X=X, Y=Y, mean=mean, inv=inv, lo=lo, hi=hi, ymean=ymean, ystd=ystd, net=net,
                flag=flag, out=out)


def run(st):
    op = st["op"]
    if op == "substeps":
        fv3.acoustic_substeps(st["s"], st["g"], st["dt"], st["n_split"])
    elif op == "tracers":
        fv3.tracer_transport(st["qs"], st["s"], st["g"])
    elif op == "dynamics":
        fv3.dynamics(st["s"], st["g"], st["qs"], st["ak"], st["bk"], st["dt"], st["k_split"], st["n_split"])
    elif op == "ensemble":
        st["ens"].run()
    elif op == "sums":
        return fv3.mass_sums(st["g"], st["s"].f["delp"], st["s"].f["pt"], st["qs"])
    elif op == "train":
        for k, (X, T) in enumerate(st["batches"]):
            loss = st["net"].train_step(X, T, lr=1e-3, want_loss=k == len(st["batches"]) - 1)
        return {"loss": loss, "params": st["net"].get_params()}
    else:
        st["flag"].zero_()
        fv3.column_features(st["s"], st["g"], st["mean"], st["inv"], st["X"], st["flag"], st["lo"], st["hi"])
        st["net"].forward(st["X"], st["Y"])
        fv3.apply_correction(st["s"], st["g"], st["Y"], st["ymean"], st["ystd"], 10800.0, st["flag"])
    return st["out"]


# -------------------------------------------------------------------- work
def _cells(kind, n, nz):
    return (6 if kind == 1 else 1) * n * n * nz


def work(case):
    """Bytes and operations a pass cannot do without.  A substep reads the six
    prognostics and the accumulators and writes them back with the C-grid
    winds and the interface fields (the substeps of one pass depend on each
    other through whole fields that fit no cache); the operations are a count
    of the scheme's, about 1300 per cell and substep, 300 per cell and tracer
    sub-cycle, 120 per remapped field and cell."""
    op = case["op"]
    eb = 4 if case.get("precision") == "mixed" else 8
    substep = 2 * (7 * eb + 24) + 2 * eb + 16   # u v w delp pt cx cy | delz mfx mfy; uc vc; pfull phi
    if op == "substeps":
        c = _cells(case["kind"], case["n"], case["nz"]) * case["n_split"]
        return {"bytes": c * substep, "flops": c * 1300.0}
    if op == "tracers":
        c = _cells(case["kind"], case["n"], case["nz"])
        return {"bytes": c * (2 * eb * case["nq"] + 2 * eb + 24), "flops": c * case["nq"] * 300.0}
    if op == "dynamics":
        c, k, q = _cells(case["kind"], case["n"], case["nz"]), case["k_split"], case["nq"]
        return {"bytes": c * k * (case["n_split"] * substep + 4 * eb * q + 2 * (5 * eb + 8)),
                "flops": c * k * (1300.0 * case["n_split"] + 300.0 * q + 120.0 * (5 + q))}
    if op == "ensemble":
        sizes, m = np.random.default_rng(4), case["members"]
        ns = sizes.integers(case["n_lo"], case["n_hi"] + 1, m)
        nzs = sizes.integers(case["nz_lo"], case["nz_hi"] + 1, m)
        c = float((ns * ns * nzs).sum()) * case["n_split"]
        return {"bytes": c * substep, "flops": c * 1300.0}
    if op == "sums":
        c = _cells(case["kind"], case["n"], case["nz"])
        return {"bytes": c * eb * (2 + case["nq"]), "flops": c * 10.0 * (2 + case["nq"])}
    h, i, o = case["hidden"], 5 * case["nz"], 3 * case["nz"]
    p = i * h + h * h + h * o
    if op == "train":
        b, r = case["batches"], case["rows"]
        return {"bytes": b * (4.0 * r * (i + o) + 24.0 * p) + 4.0 * p, "flops": 6.0 * b * r * p}
    r = 6 * case["n"] ** 2
    return {"bytes": r * (5.0 * eb * case["nz"] + 4 * i + 4 * o + 6 * eb * case["nz"]), "flops": 2.0 * r * p}


# ------------------------------------------------------------------- exact
def _areas(kind, n):
    if kind == 0:
        return torch.full((1, n, n), 1.0e6, dtype=torch.float64, device="cuda")
    B = _corners(n)
    quad = (B[:, :-1, :-1], B[:, :-1, 1:], B[:, 1:, 1:], B[:, 1:, :-1])

    def excess(a, b, c):   # spherical triangle
        num = (a * torch.linalg.cross(b, c)).sum(-1).abs()
        return 2 * torch.atan2(num, 1 + (a * b).sum(-1) + (b * c).sum(-1) + (c * a).sum(-1))

    return RADIUS ** 2 * (excess(quad[0], quad[1], quad[2]) + excess(quad[0], quad[2], quad[3]))


def _bf(x):
    """The network's operands are BF16 by definition of the entry point."""
    return x.float().bfloat16().double()


def _net(P, X):
    """Activations of the three layers in 64 bits (operands rounded as the entry point says)."""
    h1 = torch.tanh(_bf(X) @ _bf(P[0]) + P[1])
    h2 = torch.tanh(_bf(h1) @ _bf(P[2]) + P[3])
    return h1, h2, _bf(h2) @ _bf(P[4]) + P[5]


def _exact_train(case, seed):
    P = [torch.from_numpy(p).cuda().double() for p in _net_params(case, seed)]
    m, v = [torch.zeros_like(p) for p in P], [torch.zeros_like(p) for p in P]
    for k, (X, T) in enumerate(_batches(case, seed)):
        h1, h2, Y = _net(P, X)
        loss = ((Y - T.double()) ** 2).mean()
        dY = 2.0 / T.numel() * (Y - T.double())
        dZ2 = (_bf(dY) @ _bf(P[4]).T) * (1 - h2 ** 2)
        dZ1 = (_bf(dZ2) @ _bf(P[2]).T) * (1 - h1 ** 2)
        G = [_bf(X).T @ _bf(dZ1), dZ1.sum(0), _bf(h1).T @ _bf(dZ2), dZ2.sum(0), _bf(h2).T @ _bf(dY), dY.sum(0)]
        for q in range(6):
            m[q] = 0.9 * m[q] + 0.1 * G[q]
            v[q] = 0.999 * v[q] + 0.001 * G[q] ** 2
            mh, vh = m[q] / (1 - 0.9 ** (k + 1)), v[q] / (1 - 0.999 ** (k + 1))
            P[q] = P[q] - 1e-3 * mh / (vh.sqrt() + 1e-8)
    return {"loss": float(loss), "params": P}


def exact(case, seed):
    """64-bit values where they follow from the inputs by a few lines; the
    dynamical core's own fields have none here (None)."""
    op = case["op"]
    if op == "train":
        return _exact_train(case, seed)
    if op == "sums":
        st = prepare(case, seed)
        g, n = st["g"], case["n"]
        m = _interior(g, st["s"].f["delp"]).double() * _areas(case["kind"], n)[:, None]
        return np.array([float(m.sum())] + [float((_interior(g, f).double() * m).sum())
                                            for f in [st["s"].f["pt"]] + st["qs"]])
    if op == "correct":
        st = prepare(case, seed)
        g, s, nz, n = st["g"], st["s"], case["nz"], case["n"]
        u, v = (_views(g, s, (k,))[k].double() for k in ("u", "v"))
        cells = [0.5 * (u[:, :, :-1] + u[:, :, 1:]), 0.5 * (v[..., :-1] + v[..., 1:])]
        cells += [_interior(g, s.f[k]).double() for k in ("pt", "w", "delp")]
        cols = torch.cat([c.permute(0, 2, 3, 1).reshape(-1, nz) for c in cells], 1)
        X = (cols - st["mean"].double()) * st["inv"].double()
        P = [torch.from_numpy(p).cuda().double() for p in _net_params(case, seed)]
        Y = _net(P, X)[2]
        dpt = 10800.0 * (Y[:, 2 * nz:] * st["ystd"][2 * nz:].double() + st["ymean"][2 * nz:].double())
        pt = cells[2] + dpt.reshape(6, n, n, nz).permute(0, 3, 1, 2)
        return {"u": None, "v": None, "pt": pt, "X": X, "Y": Y, "flag": None}
    return None
