"""The calls this library is timed on.

A staggered RHMC program spends its time in multi-shift solves, in the Dirac
operator inside them, and in the forces and link updates between them; a
measurement program solves on stored configurations, one lattice at a time, in
mixed precision, or many small lattices at once; a learned force model is
trained and applied on the links.  Each case is one such call through the
Python binding, on the lattice sizes of this repository's tests and benchmark
(4^4 to 48^3x12, also extents that no tile divides), with the masses, tables
and tolerances used there.

Links are U = exp(i eps H), H = sum_a h_a lambda_a / 2 with h_a ~ N(0, 1):
eps = 0.2 is the smooth field of the benchmark's solves, eps = 0.5 has the
plaquette (about 0.5) of the thermalised 16^3x8 chain and needs its hundreds of
CG iterations.  Vectors are handed over in the library's internal form (a half
vector is [colour][site], a momentum [parity][mu][a][site]), as a program keeps
them between calls; gauge fields go in and out in the canonical form.
"""
import json
import math
import os

import numpy as np
import torch

from paper_1710_09178_amd import stag

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAXITER = 100000


# ---------------------------------------------------------------------------
# the cases
def _dims(nx, ny, nz, nt):
    return {"nx": nx, "ny": ny, "nz": nz, "nt": nt}


def listed():
    return [
        # one operator application on the smallest test lattice: a call's fixed cost
        {"name": "operator_4c4", "kind": "operator", **_dims(4, 4, 4, 4), "eps": 0.3, "mass": 0.1,
         "links": "f64_18", "naik": False},
        # the operator where the links (764 MB) stay in no cache
        {"name": "operator_48c3x12", "kind": "operator", **_dims(48, 48, 48, 12), "eps": 0.2, "mass": 0.005,
         "links": "f64_18", "naik": False},
        # a short solve on a small lattice (heat bath or action of a test-sized RHMC)
        {"name": "solve_8c4", "kind": "solve", **_dims(8, 8, 8, 8), "eps": 0.2, "mass": 0.1, "table": "xm050_n8_m0.1",
         "tol": 1e-10, "links": "f64_18", "naik": False},
        # the action solve of the 16^3x8 RHMC: 20 poles, thermal links, hundreds of iterations
        {"name": "solve_16c3x8_hot", "kind": "solve", **_dims(16, 16, 16, 8), "eps": 0.5, "mass": 0.02,
         "table": "xm050_n20_m0.02", "tol": 1e-12, "links": "f64_18", "naik": False},
        # the benchmark's solve: 12 poles of x^(-1/4), m 0.005, all solutions kept
        {"name": "solve_32c3x8", "kind": "solve", **_dims(32, 32, 32, 8), "eps": 0.2, "mass": 0.005,
         "table": "xm025_n12_m0.005", "tol": 1e-10, "links": "f64_18", "naik": False},
        # the improved operator with 12-real links, extents that no tile or XCD slab divides
        {"name": "solve_18x14x10x12_naik", "kind": "solve", **_dims(18, 14, 10, 12), "eps": 0.2, "mass": 0.02,
         "table": "xm050_n12_m0.02_h88", "tol": 1e-10, "links": "f64_12", "naik": True},
        # the precision form: FP32 Krylov vectors, refined to the FP64 residual
        {"name": "mixed_24c3x6", "kind": "mixed", **_dims(24, 24, 24, 6), "eps": 0.2, "mass": 0.02,
         "table": "xp025_n12_m0.02", "tol": 1e-11, "sloppy": "f32_18"},
        # one pseudofermion force of the 16^3x8 molecular dynamics, solve and all
        {"name": "force_16c3x8_hot", "kind": "force", **_dims(16, 16, 16, 8), "eps": 0.5, "mass": 0.02,
         "table": "xm050_n12_m0.02", "tol": 1e-11, "links": "f64_18", "naik": False},
        # a gauge step on a stored configuration: load it, Wilson force, momentum and
        # link update, plaquette, write it back
        {"name": "gauge_step_32c3x8", "kind": "gauge_step", **_dims(32, 32, 32, 8), "eps": 0.5, "beta": 5.4, "dt": 0.05},
        # measurement solves on many small lattices at once, 4 sources each
        {"name": "batch_3x8c4_3x12c3x6_3x16c3x8", "kind": "batch", "lattices": "8.8.8.8 12.12.12.6 16.16.16.8", "copies": 3,
         "nrhs": 4, "eps": 0.2, "table": "xm025_n12_m0.005", "tol": 1e-10},
        # the learned force: one epoch over stored pairs, then the force on the links
        {"name": "model_16c3x8", "kind": "model", **_dims(16, 16, 16, 8), "eps": 0.5, "pairs": 4},
        # a whole RHMC trajectory of the 16^3x8 chain (5 of its 20 leapfrog steps)
        {"name": "trajectory_16c3x8_hot", "kind": "trajectory", **_dims(16, 16, 16, 8), "eps": 0.5, "mass": 0.02,
         "beta": 5.4, "n_steps": 5, "dt": 0.05},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_dims(rng, lo, hi):
    """Even extents 4..32 whose volume is near a log-uniform draw of [lo, hi]."""
    want = _log(rng, lo, hi)
    while True:
        d = [2 * rng.randint(2, 16) for _ in range(3)]
        nt = 2 * round(want / (d[0] * d[1] * d[2]) / 2)
        if 4 <= nt <= 32 and lo <= d[0] * d[1] * d[2] * nt <= hi:
            return _dims(*d, nt)


def draw(rng):
    kind = rng.choices(["operator", "solve", "mixed", "force", "gauge_step", "batch", "model", "trajectory"],
                       [2, 4, 1, 2, 1, 1, 1, 1])[0]
    fmt = rng.choice(["f64_18", "f64_18", "f64_12"])
    naik = rng.random() < 0.25
    if kind == "operator":
        links = rng.choice(["f64_18", "f64_18", "f64_12", "f32_18", "f16_12"])
        return {"kind": kind, **_draw_dims(rng, 256, 500000), "eps": rng.choice([0.2, 0.5]),
                "mass": round(_log(rng, 0.005, 0.1), 4), "links": links, "naik": naik}
    if kind in ("solve", "force"):
        table = "xm050_n12_m0.02_h88" if naik else rng.choice(
            ["xm050_n12_m0.02", "xm050_n20_m0.02", "xp025_n12_m0.02"] if kind == "solve" else ["xm050_n12_m0.02"])
        return {"kind": kind, **_draw_dims(rng, 256, 250000), "eps": 0.2, "mass": 0.02, "table": table, "tol": 1e-10,
                "links": fmt, "naik": naik}
    if kind == "mixed":
        return {"kind": kind, **_draw_dims(rng, 1000, 100000), "eps": 0.2, "mass": 0.02, "table": "xp025_n12_m0.02",
                "tol": 1e-11, "sloppy": rng.choice(["f32_18", "f16_12"])}
    if kind == "gauge_step":
        return {"kind": kind, **_draw_dims(rng, 256, 250000), "eps": 0.5, "beta": round(rng.uniform(5.2, 5.7), 2),
                "dt": round(rng.uniform(0.02, 0.1), 3)}
    if kind == "batch":
        shapes = rng.sample(["4.4.4.4", "8.8.8.8", "8.6.4.10", "12.12.12.6", "16.16.16.8", "10.8.12.6"], rng.randint(2, 4))
        return {"kind": kind, "lattices": " ".join(shapes), "copies": rng.randint(1, 3), "nrhs": rng.randint(1, 4),
                "eps": 0.2, "table": "xm025_n12_m0.005", "tol": 1e-10}
    if kind == "model":
        return {"kind": kind, **_draw_dims(rng, 1000, 60000), "eps": 0.5, "pairs": rng.randint(1, 4)}
    return {"kind": kind, **_draw_dims(rng, 256, 30000), "eps": 0.2, "mass": 0.02, "beta": 5.4,
            "n_steps": rng.randint(1, 4), "dt": 0.05}


# ---------------------------------------------------------------------------
# inputs
_FMT = {"f64_18": stag.LINKS_F64_18, "f64_12": stag.LINKS_F64_12, "f32_18": stag.LINKS_F32_18,
        "f16_12": stag.LINKS_F16_12}
_SLOPPY = ("f32_18", "f16_12")


def _case_dims(case):
    return case["nx"], case["ny"], case["nz"], case["nt"]


def _table(name):
    with open(os.path.join(ROOT, "synth", "rational", name + ".json")) as f:
        return json.load(f)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _mm(a, b):
    """3x3 products of complex fields [..., 3, 3], elementwise."""
    c = a[..., :, 0:1] * b[..., 0:1, :]
    c = c + a[..., :, 1:2] * b[..., 1:2, :]
    return c + a[..., :, 2:3] * b[..., 2:3, :]


def _dag(a):
    return a.conj().transpose(-1, -2)


def _algebra(p):
    """sum_a p_a lambda_a / 2 for real coordinates p [..., 8]."""
    h, r3 = 0.5, 1.0 / math.sqrt(3.0)
    X = torch.zeros(p.shape[:-1] + (3, 3), dtype=torch.complex128, device=p.device)
    X[..., 0, 0] = h * (p[..., 2] + r3 * p[..., 7])
    X[..., 1, 1] = h * (-p[..., 2] + r3 * p[..., 7])
    X[..., 2, 2] = -2 * h * r3 * p[..., 7]
    for (i, j), (a, b) in (((0, 1), (0, 1)), ((0, 2), (3, 4)), ((1, 2), (5, 6))):
        X[..., i, j] = h * torch.complex(p[..., a], -p[..., b])
        X[..., j, i] = h * torch.complex(p[..., a], p[..., b])
    return X


def _su3(u):
    """Gram-Schmidt of rows 0 and 1, row 2 = conj(row 0 x row 1)."""
    r0 = u[..., 0, :] / u[..., 0, :].abs().square().sum(-1, keepdim=True).sqrt()
    r1 = u[..., 1, :] - (r0.conj() * u[..., 1, :]).sum(-1, keepdim=True) * r0
    r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
    return torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj()], -2)


def _expi(X):
    """exp(i X) of Hermitian X: Taylor series of X / 2^8, squared 8 times."""
    Z = X * (1j / 256.0)
    one = torch.eye(3, dtype=torch.complex128, device=X.device)
    E = one + Z / 9
    for k in range(8, 0, -1):
        E = one + _mm(Z, E) / k
    for _ in range(8):
        E = _mm(E, E)
    return E


def _links(dims, eps, gen):
    nx, ny, nz, nt = dims
    h = torch.randn((nt, nz, ny, nx, 4, 8), generator=gen, device="cuda", dtype=torch.float64)
    return _su3(_expi(_algebra(eps * h))).contiguous()


def _source(dims, gen):
    """A Gaussian even half vector, [site][colour] complex."""
    nx, ny, nz, nt = dims
    v = torch.randn((nx * ny * nz * nt // 2, 3, 2), generator=gen, device="cuda", dtype=torch.float64)
    return torch.view_as_complex(v)


def _momentum(dims, gen):
    nx, ny, nz, nt = dims
    return torch.randn((nt, nz, ny, nx, 4, 8), generator=gen, device="cuda", dtype=torch.float64)


def _batch_dims(case):
    one = [tuple(int(v) for v in d.split(".")) for d in case["lattices"].split()]
    return [d for d in one for _ in range(case["copies"])]


def _batch_inputs(case, seed):
    g = _generator(seed)
    dims = _batch_dims(case)
    U = [_links(d, case["eps"], g) for d in dims]
    b = [_source(d, g) for d in dims for _ in range(case["nrhs"])]
    masses = np.random.default_rng(int(seed)).uniform(0.005, 0.05, len(dims)).tolist()
    return dims, U, b, masses


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        dims, U, b, masses = _batch_inputs(case, seed)
        B = stag.Batch(dims, case["nrhs"])
        for i, u in enumerate(U):
            B.set_gauge(i, u)
        return {"kind": kind, "B": B, "masses": masses, "rat": _table(case["table"]), "tol": case["tol"],
                "b": torch.cat([v.reshape(-1) for v in b])}
    g = _generator(seed)
    dims = _case_dims(case)
    lat = stag.Lattice(dims)
    U = _links(dims, case["eps"], g)
    lat.set_gauge(U)
    s = {"kind": kind, "lat": lat}
    if kind in ("operator", "solve", "mixed", "force"):
        s["mass"] = case["mass"]
        s["b"] = lat.vec_import(_source(dims, g), 0)
        if case.get("naik"):
            lat.set_naik()
        if case.get("links") == "f64_12":
            lat.set_link_format(stag.LINKS_F64_12)
    if kind == "operator":
        s["out"] = lat.new_vec()
        s["fmt"] = _FMT[case["links"]] if case["links"] in _SLOPPY else None
    elif kind in ("solve", "mixed"):
        s.update(rat=_table(case["table"]), tol=case["tol"])
        s["xs"] = [lat.new_vec() for _ in s["rat"]["pole"]]
        s["sum"] = lat.new_vec()
        s["sloppy"] = _FMT[case["sloppy"]] if kind == "mixed" else None
    elif kind == "force":
        s.update(rat=_table(case["table"]), tol=case["tol"], mom=lat.new_mom())
    elif kind == "gauge_step":
        s.update(U=U, p=lat.mom_import(_momentum(dims, g)), mom=lat.new_mom(), beta=case["beta"], dt=case["dt"])
    elif kind == "model":
        sur = stag.Surrogate(lat, case["pairs"], seed=3)
        mom = lat.new_mom()
        for k in range(case["pairs"]):
            # stand-ins of recorded pairs: links of the same ensemble, Gauss-like targets
            lat.set_gauge(_links(dims, case["eps"], g))
            lat.gauge_force(5.4, mom, 0.0)
            target = lat.mom_import(_momentum(dims, g)) + mom
            torch.cuda.synchronize()
            sur.add_pair(target)
        lat.set_gauge(U)
        s.update(sur=sur, p0=sur.get_params(), mom=mom)
    elif kind == "trajectory":
        s.update(U=U, mom=lat.mom_import(_momentum(dims, g)),
                 xi=lat.vec_import(_source(dims, g) * math.sqrt(0.5), 0), beta=case["beta"], mass=case["mass"],
                 n_steps=case["n_steps"], tau=case["dt"] * case["n_steps"], md=_table("xm050_n12_m0.02"),
                 action=_table("xm050_n20_m0.02"), heatbath=_table("xp025_n20_m0.02"))
    return s


# ---------------------------------------------------------------------------
# one pass
def run(s):
    kind, lat = s["kind"], s.get("lat")
    if kind == "operator":
        if s["fmt"] is None:
            lat.mdagm(s["out"], s["b"], s["mass"])
        else:
            lat.mdagm_sloppy(s["out"], s["b"], s["mass"], s["fmt"])
        return s["out"]
    if kind == "solve":
        lat.multishift_solve(s["mass"], s["rat"], s["tol"], MAXITER, s["b"], s["xs"], s["sum"], true_resid=False)
        return {"x": s["xs"], "sum": s["sum"]}
    if kind == "mixed":
        lat.multishift_solve_mixed(s["mass"], s["rat"], s["tol"], MAXITER, s["b"], s["xs"], sloppy=s["sloppy"],
                                   true_resid=False)
        return {"x": s["xs"]}
    if kind == "force":
        lat.fermion_force(s["mass"], s["rat"], s["tol"], MAXITER, s["b"], s["mom"], 0.0)
        return s["mom"]
    if kind == "gauge_step":
        lat.set_gauge(s["U"])
        s["mom"].copy_(s["p"])
        lat.gauge_force(s["beta"], s["mom"], s["dt"])
        lat.link_update(s["mom"], s["dt"])
        action, plaquette = lat.gauge_action(s["beta"])
        return {"links": lat.get_gauge(), "mom": s["mom"], "action": action, "plaquette": plaquette}
    if kind == "batch":
        x, _ = s["B"].solve(s["masses"], s["rat"], s["b"], tol=s["tol"], maxiter=MAXITER, true_resid=False)
        return x
    if kind == "model":
        s["sur"].set_params(s["p0"])
        loss = s["sur"].train(1, 1e-3)
        s["sur"].force(s["mom"], 0.0)
        return {"loss": loss, "params": s["sur"].get_params(), "force": s["mom"]}
    lat.set_gauge(s["U"])
    info = lat.trajectory(s["beta"], s["mass"], s["tau"], s["n_steps"], s["md"], s["action"], s["heatbath"],
                          tol_md=1e-11, tol_action=1e-11, inject_mom=s["mom"], inject_xi=s["xi"], inject_u=0.0)
    out = {k: info[k] for k in ("K_old", "Sg_old", "Sf_old", "K_new", "Sg_new", "Sf_new", "plaquette")}
    out["links"] = lat.get_gauge()
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
def _iterations(case, mass, tol):
    """CG iterations of the lightest shift, 0.5 sqrt(cond) ln(2 / tol); the smallest
    eigenvalue of A is 4 m^2 plus what the lowest momentum of the antiperiodic time
    direction gives on smooth links, and about 0.045 on the rough ones."""
    if "nt" in case:
        nt = case["nt"]
    else:
        nt = max(d[3] for d in _batch_dims(case))
    lo = 4 * mass * mass + (4 * math.sin(math.pi / nt) ** 2 * 0.5 if case["eps"] < 0.3 else 0.045)
    return 0.5 * math.sqrt(60.0 / lo) * math.log(2 / tol) * 0.5


def work(case):
    kind = case["kind"]
    if kind == "batch":
        vh = sum(math.prod(d) // 2 for d in _batch_dims(case))
        n = len(_table(case["table"])["pole"])
        it = _iterations(case, 0.02, case["tol"])
        return {"bytes": vh * (1152.0 + 48 * case["nrhs"] * (1 + n)),
                "flops": vh * case["nrhs"] * it * (2 * 570.0 + 72 + 48 * n)}
    vh = math.prod(_case_dims(case)) // 2
    link = {"f64_12": 96, "f32_18": 72, "f16_12": 24}.get(case.get("links"), 144)
    stencil = 1146.0 if case.get("naik") else 570.0
    per_links = 8.0 * link * (2 if case.get("naik") else 1)  # a parity's worth of links, per site
    if kind == "operator":
        # both hops read every link; the intermediate vector stays on the chip
        return {"bytes": vh * (per_links + 96), "flops": vh * (2 * stencil + 12)}
    if kind in ("solve", "mixed", "force"):
        n = len(_table(case["table"])["pole"])
        it = _iterations(case, case["mass"], case["tol"])
        out = 512.0 if kind == "force" else 48.0 * (n + 1)
        return {"bytes": vh * (per_links + 48 + out), "flops": vh * it * (2 * stencil + 72 + 48 * n)}
    if kind == "gauge_step":
        # links in and out, momenta in and out; 6 staples, exponential, plaquette
        return {"bytes": vh * 8.0 * (2 * 144 + 3 * 64), "flops": vh * 8.0 * (12 * 198 + 198 + 2000 + 500)}
    if kind == "model":
        rows = 8.0 * vh
        return {"bytes": rows * (case["pairs"] * (32 + 224 + 32) + 144 + 64 + 64),
                "flops": rows * (case["pairs"] * 37e3 + 12e3)}
    it = _iterations(case, case["mass"], 1e-11)
    return {"bytes": vh * (8.0 * 144 * 2 + 512 + 48),
            "flops": vh * (case["n_steps"] + 4) * it * (2 * 570.0 + 72 + 48 * 12)}


# ---------------------------------------------------------------------------
# the same results in plain torch, 64 bits
_AXIS = (3, 2, 1, 0)


def _coords(dims):
    nx, ny, nz, nt = dims
    t, z, y, x = torch.meshgrid(*(torch.arange(n, device="cuda") for n in (nt, nz, ny, nx)), indexing="ij")
    return x, y, z, t


class _Operator:
    """A = 4 m^2 - D_eo D_oe on full-lattice fields [t][z][y][x][colour] that vanish on odd sites."""

    def __init__(self, dims, U, mass, naik=False):
        x, y, z, t = _coords(dims)
        self.even = ((x + y + z + t) % 2 == 0).reshape(-1)
        self.dims, self.m2 = dims, 4 * mass * mass
        self.c1, self.c3 = (9.0 / 8.0, -1.0 / 24.0) if naik else (1.0, 0.0)
        sign = [torch.ones_like(x), 1 - 2 * (x % 2), 1 - 2 * ((x + y) % 2),
                (1 - 2 * ((x + y + z) % 2)) * torch.where(t == dims[3] - 1, -1, 1)]
        self.sign = [s.double() for s in sign]
        self.U = [U[..., mu, :, :] * self.sign[mu][..., None, None] for mu in range(4)]
        self.L = []
        if naik:
            for mu in range(4):
                # the phase of direction mu once, the boundary sign once per link that crosses
                b = torch.where(t == dims[3] - 1, -1.0, 1.0) if mu == 3 else torch.ones_like(self.sign[0])
                eta = self.sign[mu] * b
                W = U[..., mu, :, :] * b[..., None, None]
                W1, W2 = (torch.roll(W, -k, _AXIS[mu]) for k in (1, 2))
                self.L.append(_mm(_mm(W, W1), W2) * eta[..., None, None])

    def D(self, v):
        out = torch.zeros_like(v)
        for c, links, hop in ((self.c1, self.U, 1), (self.c3, self.L, 3)):
            for mu, u in enumerate(links):
                f = torch.roll(v, -hop, _AXIS[mu])
                out += c * (u * f[..., None, :]).sum(-1)
                out -= c * torch.roll((u.conj() * v[..., :, None]).sum(-2), hop, _AXIS[mu])
        return out

    def __call__(self, v):
        return self.m2 * v - self.D(self.D(v))

    def full(self, half):
        nx, ny, nz, nt = self.dims
        v = torch.zeros((nx * ny * nz * nt, 3), dtype=torch.complex128, device="cuda")
        v[self.even] = half
        return v.view(nt, nz, ny, nx, 3)

    def half(self, v):
        return v.reshape(-1, 3)[self.even]


def _multishift(A, b, poles, tol=1e-15):
    """(A + pole_k) x_k = b by shifted CG from the smallest pole."""
    base = min(range(len(poles)), key=lambda k: poles[k])
    shift = [p - poles[base] for p in poles]
    x = [torch.zeros_like(b) for _ in poles]
    r, p = b.clone(), [b.clone() for _ in poles]
    z, zo, a_old, b_old = [1.0] * len(poles), [1.0] * len(poles), 1.0, 0.0
    rr = float(torch.linalg.vector_norm(r)) ** 2
    stop = tol * tol * rr
    for _ in range(20000):
        live = [k for k in range(len(poles)) if z[k] * z[k] * rr > stop]
        if not live:
            break
        q = A(p[base]) + poles[base] * p[base]
        alpha = rr / float(torch.real(torch.sum(p[base].conj() * q)))
        r = r - alpha * q
        rn = float(torch.linalg.vector_norm(r)) ** 2
        beta = rn / rr
        for k in live:
            zn, q_k = 1.0, 1.0
            if k != base:
                zn = z[k] * zo[k] * a_old / (alpha * b_old * (zo[k] - z[k]) + zo[k] * a_old * (1 + shift[k] * alpha))
                q_k = zn / z[k]
            x[k] += alpha * q_k * p[k]
            p[k] = zn * r + beta * q_k * q_k * p[k]
            zo[k], z[k] = z[k], zn
        if base not in live:
            p[base] = r + beta * p[base]
        a_old, b_old, rr = alpha, beta, rn
    return x


def _internal(half):
    """[site][colour] complex to the library's [colour][site], as doubles."""
    return torch.view_as_real(half.transpose(0, 1).contiguous()).reshape(-1)


def _internal_mom(dims, P):
    """[t][z][y][x][mu][a] to the library's [parity][mu][a][site]."""
    x, y, z, t = _coords(dims)
    par = ((x + y + z + t) % 2).reshape(-1)
    flat = P.reshape(-1, 32)
    return torch.cat([flat[par == q].transpose(0, 1).reshape(-1) for q in (0, 1)])


def _im_tr(M):
    """Im tr(lambda_a M / 2) for a = 0..7."""
    e = M.imag, M.real
    f = [e[0][..., 1, 0] + e[0][..., 0, 1], e[1][..., 0, 1] - e[1][..., 1, 0], e[0][..., 0, 0] - e[0][..., 1, 1],
         e[0][..., 2, 0] + e[0][..., 0, 2], e[1][..., 0, 2] - e[1][..., 2, 0], e[0][..., 2, 1] + e[0][..., 1, 2],
         e[1][..., 1, 2] - e[1][..., 2, 1],
         (e[0][..., 0, 0] + e[0][..., 1, 1] - 2 * e[0][..., 2, 2]) / math.sqrt(3.0)]
    return 0.5 * torch.stack(f, -1)


def _exact_force(A, b, rat):
    """F_a(x, mu) = 2 sum_k c_k Im tr[T_a U_mu(x) chi_k(x + mu) chi_k(x)^dag] eps(x) (one-hop operator)."""
    dims = A.dims
    eps = torch.where(A.even, 1.0, -1.0).view(dims[3], dims[2], dims[1], dims[0])
    F = torch.zeros(eps.shape + (4, 8), dtype=torch.float64, device="cuda")
    for c, X in zip(rat["residue"], _multishift(A, b, rat["pole"])):
        chi = X + A.D(X)
        for mu in range(4):
            W = torch.roll(chi, -1, _AXIS[mu])[..., :, None] * chi.conj()[..., None, :]
            F[..., mu, :] += 2 * c * eps[..., None] * _im_tr(_mm(A.U[mu], W))
    return F


def _plaquettes(U):
    s = 0.0
    for mu in range(4):
        for nu in range(mu + 1, 4):
            a, b = U[..., mu, :, :], U[..., nu, :, :]
            P = _mm(_mm(a, torch.roll(b, -1, _AXIS[mu])), _dag(_mm(b, torch.roll(a, -1, _AXIS[nu]))))
            s += float(P.diagonal(dim1=-2, dim2=-1).real.sum())
    return s


def _exact_gauge_step(dims, U, p, beta, dt):
    F = torch.empty(p.shape, dtype=torch.float64, device="cuda")
    for mu in range(4):
        u = U[..., mu, :, :]
        S = torch.zeros_like(u)
        for nu in range(4):
            if nu != mu:
                v = U[..., nu, :, :]
                vf = torch.roll(v, -1, _AXIS[mu])
                S += _mm(_mm(vf, _dag(torch.roll(u, -1, _AXIS[nu]))), _dag(v))
                S += torch.roll(_mm(_mm(_dag(vf), _dag(u)), v), 1, _AXIS[nu])
        F[..., mu, :] = -(beta / 3) * _im_tr(_mm(u, S))
    p = p + dt * F
    U = _su3(_mm(_expi(_algebra(dt * p)), U))
    V, s = math.prod(dims), _plaquettes(U)
    return {"links": U, "mom": _internal_mom(dims, p), "action": beta * (6 * V - s / 3), "plaquette": s / (18 * V)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("model", "trajectory"):
        return None  # a bf16 network's rounding; a chain of a dozen solves and updates
    if kind == "batch":
        dims, U, b, masses = _batch_inputs(case, seed)
        rat, R = _table(case["table"]), case["nrhs"]
        cols = []
        for i, d in enumerate(dims):
            A = _Operator(d, U[i], masses[i])
            for j in range(R):
                cols.append([A.half(x).reshape(-1) for x in _multishift(A, A.full(b[i * R + j]), rat["pole"])])
        return torch.stack([torch.cat([c[k] for c in cols]) for k in range(len(rat["pole"]))])
    g = _generator(seed)
    dims = _case_dims(case)
    U = _links(dims, case["eps"], g)
    if kind == "gauge_step":
        return _exact_gauge_step(dims, U, _momentum(dims, g), case["beta"], case["dt"])
    A = _Operator(dims, U, case["mass"], bool(case.get("naik")))
    b = A.full(_source(dims, g))
    if kind == "operator":
        return _internal(A.half(A(b)))
    rat = _table(case["table"])
    if kind == "force":
        return None if case["naik"] else _internal_mom(dims, _exact_force(A, b, rat))
    x = _multishift(A, b, rat["pole"])
    if kind == "mixed":
        return {"x": [_internal(A.half(v)) for v in x]}
    total = rat["c0"] * b
    for c, v in zip(rat["residue"], x):
        total = total + c * v
    return {"x": [_internal(A.half(v)) for v in x], "sum": _internal(A.half(total))}
