"""The work that programs have this library do, for timing one version against another.

Every case goes through the Python binding as a program would: plans (and what else a program keeps) are made
once in `prepare`, `run` is one pass on fields that are on the GPU already.  Grids are tanh-stretched or
uniform, right-hand sides white noise, velocity fields a smooth swirl with noise on top, projected as a program
projects its initial state.  No tile table is loaded or tuned: the rules of the library choose the kernels.

Kinds of case:
  solve   Plan.solve of one Poisson or Helmholtz problem, in each precision and for each set of implicit directions
  batch   Batch.solve of uneven problems, replayed from a graph
  serve   requests of several grid families submitted to a Server and waited for
  ns      one Navier-Stokes time step (three substeps) in place
"""
import math
import random

import numpy as np
import torch

import paper_2603_09528_amd as tpt

# --- problems ----------------------------------------------------------------------------------------------


def _solve(name=None, n=(32, 32, 32), bc=("NN", "NN", "NN"), beta=(0.0, 0.0, 0.0), loc="CCC", kind="poisson", alpha=0.0,
           imp="xyz", prec="fp64", refine=0, nrhs=1):
    c = {"kind": "solve", "pde": kind, "alpha": alpha, "imp": imp, "prec": prec, "refine": refine, "nrhs": nrhs, "loc": loc}
    for d, k in enumerate("xyz"):
        c["n" + k], c["bc" + k], c["beta" + k] = n[d], bc[d], 0.0 if bc[d] == "PP" else beta[d]
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest call: a cavity for a regression test or a coarse level, bound by launches and latency
        _solve("cavity32", (32, 32, 32), ("NN", "NN", "NN"), (1.5, 1.5, 1.5)),
        # the pressure solve of a channel: x by real FFT, y by products with its eigenbasis
        _solve("channel256", (256, 256, 256), ("PP", "NN", "NN"), (0.0, 2.0, 2.0)),
        # a triply periodic box (homogeneous turbulence): fast transforms in x and y, cyclic lines in z
        _solve("box256", (256, 256, 256), ("PP", "PP", "PP")),
        # implicit diffusion of the wall-normal velocity of a channel: unknowns on 383 interior faces in y
        _solve("diffusion_v", (512, 384, 256), ("PP", "DD", "DD"), (0.0, 2.0, 2.0), "CFC", "helmholtz", 1e-4),
        # a duct or room stretched in every direction, sizes that are no power of two: products in x and y
        _solve("duct", (448, 320, 288), ("NN", "NN", "DD"), (2.0, 1.7, 2.2)),
        # the same diffusion step in split BF16 with two FP64 corrections, dense in x and y (three walls)
        _solve("diffusion_bf16x3", (448, 384, 256), ("DD", "DD", "DD"), (2.0, 2.0, 2.0), "CCC", "helmholtz", 1e-4, prec="bf16x3",
               refine=2),
        # a solve with FP32 transforms, an open boundary (no mirror symmetry in z), two corrections
        _solve("family320_fp32", (320, 320, 320), ("DD", "NN", "ND"), (1.2, 1.2, 1.2), prec="fp32", refine=2),
        # the largest: a uniform 1024^3 grid, fast transforms in x and y
        _solve("uniform1024", (1024, 1024, 1024), ("PP", "NN", "NN")),
        # sixteen uneven problems at once, as an ensemble or a domain decomposition has them
        {"name": "batch16", "kind": "batch", "count": 16, "lo": 48, "hi": 192, "prec": "fp64", "refine": 0, "draw": 4},
        # ten requests of four grid families to the serving loop
        {"name": "serve10", "kind": "serve", "count": 10, "families": 4, "lo": 64, "hi": 256, "prec": "fp64", "refine": 0, "draw": 5},
        # a time step of a channel with explicit diffusion, uniform in x
        {"name": "ns_explicit", "kind": "ns", "nx": 512, "ny": 256, "nz": 256, "bcx": "PP", "bcy": "NN", "bcz": "NN", "betax": 0.0,
         "betay": 2.0, "betaz": 2.0, "imp": "none", "nu": 1e-4},
        # a time step of a duct with implicit diffusion in all directions: three Helmholtz solves a substep
        {"name": "ns_implicit", "kind": "ns", "nx": 192, "ny": 160, "nz": 128, "bcx": "PP", "bcy": "NN", "bcz": "NN", "betax": 0.0,
         "betay": 2.0, "betaz": 2.0, "imp": "xyz", "nu": 1e-3},
    ]


MOST_UNKNOWNS = 40e6


def _size(rng, lo, hi):
    if rng.random() < 0.35:
        return 2 ** rng.randint(math.ceil(math.log2(lo)), math.floor(math.log2(hi)))
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _beta(rng):
    return 0.0 if rng.random() < 0.3 else round(rng.uniform(0.5, 2.5), 3)


def draw(rng):
    what = rng.random()
    if what < 0.6:
        while True:
            n = tuple(_size(rng, 24, 640) for _ in range(3))
            if n[0] * n[1] * n[2] <= MOST_UNKNOWNS:
                break
        prec = rng.choice(("fp64", "fp64", "fp64", "fp32", "bf16x3"))
        bc = [rng.choice(("PP", "NN", "DD", "ND")) for _ in range(2)] + [rng.choice(("NN", "DD", "ND", "PP"))]
        beta = [_beta(rng) for _ in range(3)]
        if prec == "fp64" and rng.random() < 0.5:
            return _solve(None, n, bc, beta, nrhs=rng.choice((1, 1, 1, 2)))
        # implicit diffusion; in the mixed modes too, where a singular problem has its constant only to the first solve's precision
        bc = [rng.choice(("PP", "DD")) for _ in range(3)]
        loc = rng.choice(("FCC", "CFC", "CCF", "CCC"))
        imp = rng.choice(("xyz", "xyz", "yz", "z")) if prec == "fp64" else "xyz"
        return _solve(None, n, bc, beta, loc, "helmholtz", round(10 ** rng.uniform(-5, -3), 7), imp, prec, 0 if prec == "fp64" else 2)
    if what < 0.85:
        kind = "batch" if what < 0.75 else "serve"
        prec = rng.choice(("fp64", "fp64", "fp32"))
        lo = rng.randint(24, 64)
        c = {"kind": kind, "count": rng.randint(4, 20), "lo": lo, "hi": rng.randint(lo + 32, 192), "prec": prec,
             "refine": 0 if prec == "fp64" else 2, "draw": rng.randint(0, 1 << 20)}
        return {**c, "families": rng.randint(2, 5)} if kind == "serve" else c
    c = {"kind": "ns", "imp": rng.choice(("none", "z", "yz", "xyz")), "nu": round(10 ** rng.uniform(-4, -2.5), 6)}
    for k in "xyz":
        c["n" + k] = _size(rng, 32, 256)
        c["bc" + k] = rng.choice(("PP", "NN")) if k != "z" else rng.choice(("NN", "NN", "PP"))
        c["beta" + k] = 0.0 if c["bc" + k] == "PP" else _beta(rng)
    return c


def _faces(n, beta):
    xi = np.arange(n + 1) / n
    x = xi if beta == 0.0 else 0.5 * (1.0 + np.tanh(beta * (xi - 0.5)) / np.tanh(0.5 * beta))
    x[0], x[-1] = 0.0, 1.0
    return x


class Problem:
    """Cells, faces, boundary conditions, locations and operator of one problem."""

    def __init__(self, n, bc, beta, loc="CCC", kind="poisson", alpha=0.0, imp="xyz"):
        self.n, self.bc, self.kind, self.alpha, self.imp = tuple(n), tuple(bc), kind, alpha, imp
        self.faces = [_faces(n[d], beta[d]) for d in range(3)]
        self.loc = tuple(loc)
        self.shape = tuple(n[d] - 1 if loc[d] == "F" and bc[d] == "DD" else n[d] for d in (2, 1, 0))

    @property
    def singular(self):
        return self.kind == "poisson" and all(b in ("PP", "NN") for b in self.bc)

    def plan(self, prec, refine, nrhs=1):
        more = {} if prec == "fp64" else {"fixed_refine": refine}
        return tpt.Plan(self.n, self.faces, self.bc, self.loc, self.kind, self.alpha, precision=prec, nrhs=nrhs, implicit=self.imp, **more)

    def rhs(self, seed, nrhs=1):
        """White noise; with no share that a singular operator cannot reach."""
        g = torch.Generator(device="cuda").manual_seed(seed)
        f = torch.randn((nrhs,) + self.shape, generator=g, dtype=torch.float64, device="cuda")
        if self.singular:
            vol = [torch.from_numpy(np.diff(x)).cuda() for x in self.faces]
            wf = torch.matmul(torch.matmul(f, vol[0]), vol[1])  # the weighted sum of each plane
            f -= (torch.matmul(wf, vol[2]) / (vol[0].sum() * vol[1].sum() * vol[2].sum())).view(-1, 1, 1, 1)
        return f[0] if nrhs == 1 else f


def _triple(c, key):
    return tuple(c[key + k] for k in "xyz")


def _problem(c):
    return Problem(_triple(c, "n"), _triple(c, "bc"), _triple(c, "beta"), c["loc"], c["pde"], c["alpha"], c["imp"])


def _uneven(c):
    """The problems of a batch, or the requests of a serving case (their families repeat)."""
    rng = random.Random(c["draw"])
    zs = ("NN", "DD", "ND") if c["prec"] == "fp64" else ("DD", "ND")  # mixed modes: no singular problems, as in draw()

    def one():
        beta = rng.uniform(0.0, 2.5)
        bc = (rng.choice(("PP", "NN", "DD", "ND")), rng.choice(("PP", "NN", "DD", "ND")), rng.choice(zs))
        if c["kind"] == "serve":  # cubic families
            n = (int(round(c["lo"] * (c["hi"] / c["lo"]) ** rng.random())),) * 3
        else:
            n = tuple(rng.randint(c["lo"], c["hi"]) for _ in range(3))
        return Problem(n, bc, [0.0 if b == "PP" else beta for b in bc])

    if c["kind"] == "batch":
        return [one() for _ in range(c["count"])]
    fams = [one() for _ in range(c["families"])]
    return [fams[0 if i == 0 else rng.randrange(len(fams))] for i in range(c["count"])]


# --- Navier-Stokes: the initial state and the step --------------------------------------------------------


def _pressure(c):
    return Problem(_triple(c, "n"), _triple(c, "bc"), _triple(c, "beta"))


def _velocity_shapes(p):
    nz, ny, nx = p.shape
    nf = [n if p.bc[d] == "PP" else n - 1 for d, n in enumerate((nx, ny, nz))]
    return (nz, ny, nf[0]), (nz, nf[1], nx), (nf[2], ny, nx)


def _time_step(p):
    return 0.1 * min(float(np.diff(x).min()) for x in p.faces)  # Courant number about 0.2


def _initial(p, seed):
    """u, v, w (not yet divergence-free) and the pressure."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    out = []
    for c, s in enumerate(_velocity_shapes(p)):
        k, j, i = (torch.linspace(0.0, 2.0 * math.pi, m, dtype=torch.float64, device="cuda") for m in s)
        a = ((j, k), (k, i), (i, j))[c]
        view = {id(k): (-1, 1, 1), id(j): (1, -1, 1), id(i): (1, 1, -1)}
        swirl = torch.sin(a[0]).view(view[id(a[0])]) * torch.cos(a[1]).view(view[id(a[1])])
        noise = torch.randn(s, generator=g, dtype=torch.float64, device="cuda")
        out.append((swirl + 0.1 * noise).contiguous())
    out.append(0.1 * torch.randn(p.shape, generator=g, dtype=torch.float64, device="cuda"))
    return out


# --- the interface ----------------------------------------------------------------------------------------


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        p = _problem(case)
        return {"kind": kind, "plan": p.plan(case["prec"], case["refine"], case["nrhs"]), "rhs": p.rhs(seed, case["nrhs"])}
    if kind == "batch":
        ps = _uneven(case)
        plans = [p.plan(case["prec"], case["refine"]) for p in ps]
        rhs = [p.rhs(seed * 64 + i) for i, p in enumerate(ps)]
        return {"kind": kind, "batch": tpt.Batch(plans), "rhs": rhs, "out": [torch.empty_like(f) for f in rhs]}
    if kind == "serve":
        ps = _uneven(case)
        plans = {id(p): p.plan(case["prec"], case["refine"]) for p in ps}
        rhs = [p.rhs(seed * 64 + i) for i, p in enumerate(ps)]
        return {"kind": kind, "server": tpt.Server(hbm_budget_bytes=4 << 30), "plans": [plans[id(p)] for p in ps], "rhs": rhs,
                "out": [torch.empty_like(f) for f in rhs]}
    p = _pressure(case)
    plan = p.plan("fp64", 0)
    u, v, w, q = _initial(p, seed)
    plan.project(u, v, w)
    ns = tpt.NavierStokes(plan, case["nu"], _time_step(p), case["imp"])
    return {"kind": kind, "ns": ns, "fields": (u, v, w, q), "phi": torch.empty_like(q)}


def run(state):
    kind = state["kind"]
    if kind == "solve":
        return state["plan"].solve(state["rhs"])
    if kind == "batch":
        return state["batch"].solve(state["rhs"], state["out"])
    if kind == "serve":
        srv = state["server"]
        tickets = [srv.submit(p, f, o) for p, f, o in zip(state["plans"], state["rhs"], state["out"])]
        srv.drain()
        for t in tickets:
            srv.poll(t)
        return state["out"]
    state["ns"].step(*state["fields"], phi=state["phi"])
    # the state that the next step starts from; Phi, the last substep's small increment of the pressure, is in it already
    return list(state["fields"])


def _passes_flops(p):
    """Operations of one application of the solve: products with the eigenbases of x and y (halved where the mirror symmetry of the
    direction splits its basis), or fast transforms, and the line solves."""
    nz, ny, nx = p.shape
    dof, per = nx * ny * nz, 30.0
    for d, n in ((0, nx), (1, ny)):
        if d not in {"xyz": (0, 1), "yz": (1,), "z": ()}[p.imp]:
            continue
        w = np.diff(p.faces[d])
        fast = p.bc[d] != "ND" and p.loc[d] == "C" and np.ptp(w) <= 1e-9 * w[0] and 8 <= n <= 2048 and n & (n - 1) == 0
        fast = fast or (p.bc[d] == "PP" and 8 <= n <= 2048 and n & (n - 1) == 0)
        per += 2 * (2.5 * math.log2(n) if fast else 2.0 * n if p.bc[d] == "ND" else 1.0 * n)
    return dof, dof * per


def work(case):
    kind = case["kind"]
    if kind == "solve":
        dof, fl = _passes_flops(_problem(case))
        r = 1 + case["refine"]
        # right-hand side in, solution out
        return {"bytes": 16.0 * dof * case["nrhs"], "flops": (fl * r + 20.0 * dof * (r - 1)) * case["nrhs"]}
    if kind in ("batch", "serve"):
        b = f = 0.0
        for p in _uneven(case):
            dof, fl = _passes_flops(p)
            b += 16.0 * dof
            f += fl * (1 + case["refine"]) + 20.0 * dof * case["refine"]
        return {"bytes": b, "flops": f}
    p = _pressure(case)
    dof, fl = _passes_flops(p)
    # a step: u, v, w, P in and out; flops of the solves and about 150 per cell and substep for the explicit terms
    solves = 3 * fl * (1 if case["imp"] == "none" else 4)
    return {"bytes": 64.0 * dof, "flops": solves + 450.0 * dof}


# --- the same results in plain torch, 64 bits: every direction by its dense eigenbasis --------------------


def _operator(faces, bc, loc):
    """Rows a, b, c of the second-difference operator of one direction and its control volumes."""
    w = np.diff(faces)
    if loc == "C":
        vol = w
        d = 0.5 * (w[:-1] + w[1:])
        wrap = 0.5 * (w[0] + w[-1])
        lo = np.concatenate([[wrap if bc == "PP" else w[0]], d])
        hi = np.concatenate([d, [wrap if bc == "PP" else w[-1]]])
    elif bc == "PP":
        up = np.roll(w, -1)
        vol, lo, hi = 0.5 * (w + up), w, up
    else:
        vol, lo, hi = 0.5 * (w[:-1] + w[1:]), w[:-1], w[1:]
    a, c = 1.0 / (vol * lo), 1.0 / (vol * hi)
    b = -(a + c)
    if bc != "PP":
        if loc == "C":
            b[0] += a[0] if bc[0] == "N" else -a[0]
            b[-1] += c[-1] if bc[1] == "N" else -c[-1]
        a[0] = c[-1] = 0.0
    return a, b, c, vol


def _basis(faces, bc, loc):
    """Eigenvalues, Q^-1, Q of one direction, on the GPU."""
    a, b, c, vol = _operator(faces, bc, loc)
    n = len(b)
    t = np.diag(b) + np.diag(a[1:], -1) + np.diag(c[:-1], 1)
    if bc == "PP":
        t[0, n - 1] += a[0]
        t[n - 1, 0] += c[n - 1]
    s = np.sqrt(vol)
    sym = t * s[:, None] / s[None, :]
    lam, q = np.linalg.eigh(0.5 * (sym + sym.T))
    if bc == "PP" or (bc == "NN" and loc == "C"):
        lam[-1], q[:, -1] = 0.0, s / math.sqrt(vol.sum())
    return tuple(torch.from_numpy(np.ascontiguousarray(m)).cuda() for m in (lam, q.T * s[None, :], q / s[:, None]))


def _dense_solve(p, f):
    """A u = f of one problem, f (Nz, Ny, Nx)."""
    nz, ny, nx = p.shape
    dirs = {"xyz": (0, 1, 2), "yz": (1, 2), "z": (2,)}[p.imp]
    bases = {d: _basis(p.faces[d], p.bc[d], p.loc[d]) for d in dirs}

    def apply(k, u):
        if 0 in bases:
            u = torch.matmul(u.reshape(nz * ny, nx), bases[0][k].T).view(nz, ny, nx)
        if 1 in bases:
            u = torch.stack([torch.matmul(bases[1][k], s) for s in u]) if nz <= 64 else torch.matmul(bases[1][k], u)
        return torch.matmul(bases[2][k], u.reshape(nz, ny * nx)).view(nz, ny, nx)

    u = apply(1, f)
    lam = torch.zeros((nz, ny, nx), dtype=torch.float64, device="cuda")
    for d in dirs:
        lam += bases[d][0].view([(1, 1, -1), (1, -1, 1), (-1, 1, 1)][d])
    if p.kind == "helmholtz":
        u /= lam.mul_(-p.alpha).add_(1.0)
    else:
        zero = lam == 0.0
        u /= lam.masked_fill_(zero, 1.0)
        u.masked_fill_(zero, 0.0)
    u = apply(2, u)
    if p.singular:  # zero mean over the last plane
        vx, vy = (torch.from_numpy(np.diff(p.faces[d])).cuda() for d in (0, 1))
        u -= torch.dot(torch.mv(u[-1], vx), vy) / (vx.sum() * vy.sum())
    return u


def _ax(d):
    return 2 - d


def _col(v, d):
    v = torch.from_numpy(np.ascontiguousarray(v)).cuda() if isinstance(v, np.ndarray) else v
    return v.view([(1, 1, -1), (1, -1, 1), (-1, 1, 1)][d])


def _shift(q, d, by, per):
    """q at the position by (-1 or +1) further along d: wrapped, or zero outside."""
    r = torch.roll(q, -by, _ax(d))
    if not per:
        r.select(_ax(d), r.shape[_ax(d)] - 1 if by > 0 else 0).zero_()
    return r


def _second(p, q, c, dirs):
    """The one-dimensional second differences of component c (None: of a cell-centred pressure field), summed over dirs."""
    out = torch.zeros_like(q)
    for d in dirs:
        per = p.bc[d] == "PP"
        bc = "PP" if per else "NN" if c is None else "DD"
        a, b, cc, _ = _operator(p.faces[d], bc, "F" if d == c else "C")
        out += _col(b, d) * q + _col(a, d) * _shift(q, d, -1, per) + _col(cc, d) * _shift(q, d, 1, per)
    return out


def _spacing(p, d):
    w = np.diff(p.faces[d])
    h = 0.5 * (w[:-1] + w[1:])
    return w, np.concatenate([h, [0.5 * (w[0] + w[-1])]]) if p.bc[d] == "PP" else h


def _grad(p, q, d):
    _, h = _spacing(p, d)
    m = len(h)
    return (torch.roll(q, -1, _ax(d)) - q).narrow(_ax(d), 0, m) / _col(h, d)


def _div(p, vel):
    out = torch.zeros(p.shape, dtype=torch.float64, device="cuda")
    for d in range(3):
        w, _ = _spacing(p, d)
        q, per = vel[d], p.bc[d] == "PP"
        if not per:  # the wall face carries no flux
            pad = list(q.shape)
            pad[_ax(d)] = 1
            q = torch.cat([q, q.new_zeros(pad)], _ax(d))
        out += (q - torch.roll(q, 1, _ax(d))) / _col(w, d)
    return out


def _advect(p, vel, c):
    """-div(u u) of component c: mean transported values, mass fluxes that sum the two cells' continuity."""
    q, per = vel[c], p.bc[c] == "PP"
    wc, hc = _spacing(p, c)
    m = len(hc)
    hi = 0.5 * (q + _shift(q, c, 1, per))
    lo = 0.5 * (q + _shift(q, c, -1, per))
    res = (lo * lo - hi * hi) / _col(hc, c)
    for e in range(3):
        if e == c:
            continue
        we, _ = _spacing(p, e)
        wq = vel[e] * _col(wc, c)
        flux = 0.5 * (wq + torch.roll(wq, -1, _ax(c))).narrow(_ax(c), 0, m)
        pe = p.bc[e] == "PP"
        if not pe:
            pad = list(flux.shape)
            pad[_ax(e)] = 1
            flux = torch.cat([flux, flux.new_zeros(pad)], _ax(e))
        t = 0.5 * (q + _shift(q, e, 1, pe))
        tl = 0.5 * (q + _shift(q, e, -1, pe))
        res -= (flux * t - torch.roll(flux, 1, _ax(e)) * tl) / (_col(hc, c) * _col(we, e))
    return res


def _exact_step(case, seed):
    p = _pressure(case)
    u, v, w, pr = _initial(p, seed)
    vel = [u, v, w]
    phi = _dense_solve(p, _div(p, vel))
    vel = [q - _grad(p, phi, d) for d, q in enumerate(vel)]
    dt, nu = _time_step(p), case["nu"]
    impl = {"none": (), "z": (2,), "yz": (1, 2), "xyz": (0, 1, 2)}[case["imp"]]
    expl = tuple(d for d in range(3) if d not in impl)
    bc = tuple("PP" if b == "PP" else "DD" for b in p.bc)
    beta = _triple(case, "beta")
    old = [None] * 3
    for al, be in ((8 / 15, 0.0), (5 / 12, -17 / 60), (3 / 4, -5 / 12)):
        ga = al + be
        cn = 0.5 * ga * nu * dt
        star = []
        for c in range(3):
            e = _advect(p, vel, c) + nu * _second(p, vel[c], c, expl)
            li = _second(p, vel[c], c, impl)
            s = vel[c] + dt * (al * e + ga * (nu * li - _grad(p, pr, c)))
            if be:
                s += dt * be * old[c]
            if impl:
                loc = "".join("F" if d == c else "C" for d in range(3))
                s = _dense_solve(Problem(p.n, bc, beta, loc, "helmholtz", cn, case["imp"]), s - cn * li)
            star.append(s)
            old[c] = e
        phi = _dense_solve(p, _div(p, star) / (ga * dt))
        vel = [q - ga * dt * _grad(p, phi, d) for d, q in enumerate(star)]
        pr = pr + phi - cn * _second(p, phi, None, impl)
    return vel + [pr]


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        p = _problem(case)
        f = p.rhs(seed, case["nrhs"])
        return _dense_solve(p, f) if case["nrhs"] == 1 else torch.stack([_dense_solve(p, g) for g in f])
    if kind in ("batch", "serve"):
        return [_dense_solve(p, p.rhs(seed * 64 + i)) for i, p in enumerate(_uneven(case))]
    return _exact_step(case, seed)
