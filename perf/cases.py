"""Workloads that time the framework's public entry points on one GPU.

Each case is one pass of a program that keeps a ``GMGPoisson`` handle (or
calls the differentiable ``poisson_solve``) on a streamer-shaped problem: one
filament along z with lognormal cell noise in the coefficient (max(a) is the
case's ``contrast``; 1 is a constant coefficient), plates phi = 0 / 1, unit
cube.  The kinds:

operator   y = A x - lifting on given cell values: ``GMGPoisson.apply``
solve      one solve without an initial guess: ``GMGPoisson.solve``
gradient   a step of an optimisation loop on the coefficient: renewal of the
           hierarchy, forward solve, adjoint solve, dL/da
step       the elliptic half of a time step: coefficient and right side from
           the densities, renewal, solve warm-started from the previous
           step's potential, field
autograd   ``poisson_solve`` and its backward, handle set-up included
krylov     BiCGSTAB with the same preconditioner: ``GMGPoisson.krylov_solve``

Solves stop at the library's default 1e-8, except the mixed-precision
forward solves whose potential is differenced afterwards (gradient, step):
those stop at 1e-10, since differencing multiplies what the solve leaves.
"""
import math

import torch

import paper_1812_08606_amd as gm

TOL, TOL_DIFFERENCED = 1e-8, 1e-10
PB, PT = 0.0, 1.0  # plate values
EPS, TAU = 1.0, 0.5  # eps0 / e and tau_eff of the time step
DENSITY = 50.0  # density scale: f = n_p - n_e of order 50


def _case(name, kind, nx, ny, nz, precision="mixed", contrast=1e3):
    return {"name": name, "kind": kind, "nx": nx, "ny": ny, "nz": nz, "precision": precision,
            "contrast": float(contrast)}


def listed():
    return [
        # the operator alone on the smallest odd grid the solver takes (one
        # level): call latency
        _case("operator_15x16x17", "operator", 15, 16, 17, "fp64"),
        # and where it is one pass over memory (a mesh of the solver
        # comparison): a residual check or a user's own iteration
        _case("operator_256x256x320", "operator", 256, 256, 320, "fp64", 1e4),
        # an odd grid that cannot be coarsened: renewal and direct solves
        _case("gradient_15x16x17", "gradient", 15, 16, 17),
        # the constant-coefficient problem of an explicit scheme, small: bound
        # by launches and the coarse levels
        _case("solve_64", "solve", 64, 64, 64, "mixed", 1.0),
        # differentiable call inside a training loop, set-up included
        _case("autograd_48x64x80", "autograd", 48, 64, 80, "fp64", 1e2),
        # time steps: a small one, a ragged one whose coarsest level has 11 x
        # 13 x 15 cells, and a large float64 one on a comparison mesh
        _case("step_128", "step", 128, 128, 128),
        _case("step_176x208x240", "step", 176, 208, 240),
        _case("step_256x256x320_fp64", "step", 256, 256, 320, "fp64"),
        # another Krylov method of the solver comparison
        _case("krylov_128x128x160_fp64", "krylov", 128, 128, 160, "fp64"),
        # the gradient workload, in both precisions, and the benchmark's size
        _case("gradient_256", "gradient", 256, 256, 256),
        _case("gradient_256_fp64", "gradient", 256, 256, 256, "fp64"),
        _case("gradient_512", "gradient", 512, 512, 512, "mixed", 1e4),
    ]


def draw(rng):
    """One more case of the ranges above: edges from about 8 to 384 cells
    (spread over their logarithm), each dimension a coarsest edge times a
    power of two, odd coarsest edges among them."""
    kind = rng.choice(["operator", "solve", "gradient", "gradient", "step", "step", "autograd", "krylov"])
    top = {"operator": 384, "autograd": 160, "krylov": 256}.get(kind, 384)
    edge = math.exp(rng.uniform(math.log(8), math.log(top)))
    levels = max(0, math.ceil(math.log2(edge / rng.uniform(8, 15))))
    while True:
        base = [max(3, round(edge / 2 ** levels * rng.uniform(0.8, 1.2))) for _ in range(3)]
        if base[0] * base[1] * base[2] <= 3600:
            break
        edge *= 0.97
    nx, ny, nz = (b << levels for b in base)
    precision = rng.choice(["mixed", "mixed", "fp64"])
    if kind in ("operator", "krylov"):
        precision = "fp64"
    contrast = 1.0 if rng.random() < 0.15 else round(math.exp(rng.uniform(math.log(10), math.log(3e3))), 3)
    c = _case("", kind, nx, ny, nz, precision, contrast)
    del c["name"]
    return c


# -- inputs -------------------------------------------------------------------


def _cells(case):
    return case["nx"] * case["ny"] * case["nz"]


def _centres(n):
    return (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) / n


def _profile(case, x0, y0, shift):
    """Gaussian in r around the axis (x0, y0), smooth window over z."""
    sigma = max(0.03, 1.5 / min(case["nx"], case["ny"]))
    x, y, z = _centres(case["nx"]), _centres(case["ny"]), _centres(case["nz"]) - shift

    def ramp(t):
        t = t.clamp(0.0, 1.0)
        return t * t * (3.0 - 2.0 * t)

    s = ramp((z - 0.2) / 0.05) * ramp((0.8 - z) / 0.05)
    gx = torch.exp(-((x - x0) ** 2) / (2.0 * sigma ** 2))
    gy = torch.exp(-((y - y0) ** 2) / (2.0 * sigma ** 2))
    return s[:, None, None] * gy[None, :, None] * gx[None, None, :]


def _densities(case, seed):
    """Electron and ion densities; the kappa that gives the contrast."""
    shape = (case["nz"], case["ny"], case["nx"])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.rand(2, generator=gen, dtype=torch.float64, device="cuda").tolist()
    x0, y0 = 0.45 + 0.1 * u[0], 0.45 + 0.1 * u[1]
    xi = torch.exp(0.1 * torch.randn(shape, generator=gen, dtype=torch.float64, device="cuda"))
    ne = _profile(case, x0, y0, 0.0) * xi
    np_ = 0.9 * _profile(case, x0, y0, 0.02) * xi
    kappa = (case["contrast"] - 1.0) / ne.max()
    return ne, np_, kappa, gen


def _problem(case, seed):
    """(a, f, g): coefficient, right side, and the gradient of a loss with
    respect to phi (a weighted box around the centre with noise)."""
    ne, np_, kappa, gen = _densities(case, seed)
    a = 1.0 + kappa * ne
    f = DENSITY * (np_ - ne)
    if case["contrast"] == 1.0:  # constant coefficient: a source at the centre, noise everywhere
        f = 2.0 * DENSITY * _profile(case, 0.5, 0.5, 0.0)
    f += 1e-3 * (2.0 * torch.rand(f.shape, generator=gen, dtype=torch.float64, device="cuda") - 1.0)
    g = torch.rand(f.shape, generator=gen, dtype=torch.float64, device="cuda") - 0.25
    nz, ny, nx = f.shape
    box = torch.zeros_like(g)
    box[nz * 2 // 5:nz * 3 // 5 + 1, ny * 2 // 5:ny * 3 // 5 + 1, nx * 2 // 5:nx * 3 // 5 + 1] = 1.0
    return a, f, g * box


def _step_problem(case, seed):
    """Densities of one time step and of the step before (one cell lower),
    and the keyword arguments of the assembly."""
    ne, np_, kappa, _ = _densities(case, seed)
    ne, np_ = DENSITY * ne, DENSITY * np_
    mu_e = float(kappa) / (DENSITY * TAU)
    hz = 1.0 / case["nz"]
    prm = dict(eps0_over_e=EPS, tau_eff=TAU, mu_e=0.99 * mu_e, mu_p=0.01 * mu_e,
               De=tuple(0.1 * hz * hz / TAU for _ in range(3)))
    return (ne, np_), (ne.roll(-1, 0), np_.roll(-1, 0)), prm


def prepare(case, seed):
    kind, prec = case["kind"], case["precision"]
    s = {"kind": kind, "tol": TOL_DIFFERENCED if prec == "mixed" and kind in ("gradient", "step") else TOL}
    if kind == "step":
        (ne, np_), (ne0, np0), prm = _step_problem(case, seed)
        h = gm.GMGPoisson(torch.ones_like(ne), precision=prec)
        a, f = h.assemble_elliptic(ne0, np0, **prm)
        h.update_coefficient(a)
        prev = h.solve(f, PB, PT, tol=s["tol"]).phi  # the potential of the step before
        s |= {"h": h, "ne": ne, "np": np_, "prm": prm, "prev": prev, "a": torch.empty_like(a),
              "f": torch.empty_like(f), "phi": torch.empty_like(f), "E": tuple(torch.empty_like(f) for _ in range(4))}
        return s
    a, f, g = _problem(case, seed)
    if kind == "autograd":
        return s | {"a": a.requires_grad_(True), "f": f.requires_grad_(True), "g": g, "precision": prec}
    # an optimisation loop renews the hierarchy in each pass: it starts from another coefficient
    s["h"] = gm.GMGPoisson(torch.ones_like(a) if kind == "gradient" else a, precision=prec)
    if kind == "operator":
        return s | {"x": f}
    return s | {"a": a, "f": f, "g": g}


# -- one pass -----------------------------------------------------------------


def run(s):
    kind = s["kind"]
    if kind == "operator":
        return s["h"].apply(s["x"], PB, PT)
    if kind == "solve":
        return s["h"].solve(s["f"], PB, PT, tol=s["tol"]).phi
    if kind == "krylov":
        return s["h"].krylov_solve(s["f"], PB, PT, method="bicgstab", tol=s["tol"])[0].phi
    if kind == "gradient":
        h = s["h"]
        h.update_coefficient(s["a"])
        phi = h.solve(s["f"], PB, PT, tol=s["tol"]).phi
        lam = h.solve(s["g"], 0.0, 0.0, tol=TOL).phi
        return {"phi": phi, "lam": lam, "dLda": h.face_flux_grad(phi, lam, PB, PT)}
    if kind == "step":
        h = s["h"]
        a, f = h.assemble_elliptic(s["ne"], s["np"], out=(s["a"], s["f"]), **s["prm"])
        h.update_coefficient(a)
        phi = h.solve(f, PB, PT, tol=s["tol"], x0=s["prev"], out=s["phi"]).phi
        return {"a": a, "f": f, "phi": phi, "E": h.electric_field(phi, PB, PT, out=s["E"])}
    a, f = s["a"], s["f"]
    a.grad = f.grad = None
    phi = gm.poisson_solve(f, a, PB, PT, tol=s["tol"], precision=s["precision"])
    phi.backward(s["g"])
    return {"phi": phi.detach(), "dLda": a.grad, "dLdf": f.grad}


def work(case):
    """Each input read once and each output written once (float64 fields),
    and the operations of one operator application per solve."""
    n = _cells(case)
    fields = {"operator": 3, "solve": 3, "krylov": 3, "gradient": 6, "step": 10, "autograd": 6}[case["kind"]]
    applications = {"gradient": 3, "step": 2, "autograd": 3}.get(case["kind"], 1)
    return {"bytes": 8.0 * fields * n, "flops": 20.0 * applications * n}


# -- the same in plain torch, 64 bits ------------------------------------------


def _apply(u, a, h, pb, pt):
    """A u - lifting (finite volumes, arithmetic face means, mirrored ghosts
    at the plates, no flux through the sides)."""
    y = torch.zeros_like(u)
    for d, hd in ((2, h[0]), (1, h[1]), (0, h[2])):
        n = u.shape[d]
        if n > 1:
            lo, hi = u.narrow(d, 0, n - 1), u.narrow(d, 1, n - 1)
            flux = 0.5 * (a.narrow(d, 0, n - 1) + a.narrow(d, 1, n - 1)) * (hi - lo) / (hd * hd)
            y.narrow(d, 0, n - 1).sub_(flux)
            y.narrow(d, 1, n - 1).add_(flux)
    y[0] += 2.0 * a[0] * (u[0] - pb) / (h[2] * h[2])
    y[-1] += 2.0 * a[-1] * (u[-1] - pt) / (h[2] * h[2])
    return y


def _spectral(shape):
    """Solver of the constant-coefficient problem in its eigenvectors."""
    def basis(n, plate):
        i = torch.arange(n, dtype=torch.float64, device="cuda")
        k = i + 1.0 if plate else i
        arg = math.pi * k[None, :] * (i[:, None] + 0.5) / n
        q = torch.sin(arg) if plate else torch.cos(arg)
        return q / q.norm(dim=0, keepdim=True), 4.0 * n * n * torch.sin(math.pi * k / (2.0 * n)) ** 2

    nz, ny, nx = shape
    (qz, ez), (qy, ey), (qx, ex) = basis(nz, True), basis(ny, False), basis(nx, False)
    lam = ez[:, None, None] + ey[None, :, None] + ex[None, None, :]
    qzt, qyt, qxt = (q.t().contiguous() for q in (qz, qy, qx))

    def along(v, mx, my, mz):
        v = (v.reshape(-1, nx) @ mx).reshape(nz, ny, nx)
        v = torch.matmul(my, v)
        return (mz @ v.reshape(nz, -1)).reshape(nz, ny, nx)

    return lambda r: along(along(r, qx, qyt, qzt) / lam, qxt, qy, qz)


def _solve(a, f, pb, pt):
    """Conjugate gradients to rounding, preconditioned by the
    constant-coefficient problem scaled with sqrt(a); the residual is
    recomputed and the iteration restarted until it stops falling."""
    nz, ny, nx = f.shape
    h = (1.0 / nx, 1.0 / ny, 1.0 / nz)
    inv, s = _spectral(f.shape), a.rsqrt()
    x = torch.zeros_like(f)
    first = last = None
    for _ in range(4):
        r = f - _apply(x, a, h, pb, pt)
        now = float(r.norm())
        first = now if first is None else first
        if now == 0.0 or (last is not None and now > 0.1 * last):
            break
        last = now
        e, p, rz = torch.zeros_like(f), None, None
        for _ in range(600):
            z = s * inv(s * r)
            rz0, rz = rz, float((r * z).sum())
            p = z if p is None else z + (rz / rz0) * p
            q = _apply(p, a, h, 0.0, 0.0)
            alpha = rz / float((p * q).sum())
            e += alpha * p
            r -= alpha * q
            if float(r.norm()) < 1e-14 * first:
                break
        x += e
    return x


def _dlda(phi, lam, h, pb, pt):
    out = torch.zeros_like(phi)
    for d, hd in ((2, h[0]), (1, h[1]), (0, h[2])):
        n = phi.shape[d]
        if n > 1:
            t = phi.diff(dim=d) * lam.diff(dim=d) / (hd * hd)
            out.narrow(d, 0, n - 1).sub_(0.5 * t)
            out.narrow(d, 1, n - 1).sub_(0.5 * t)
    out[0] -= 2.0 * (phi[0] - pb) * lam[0] / (h[2] * h[2])
    out[-1] -= 2.0 * (phi[-1] - pt) * lam[-1] / (h[2] * h[2])
    return out


def _assemble(ne, np_, prm, h):
    a = prm["eps0_over_e"] + prm["tau_eff"] * (prm["mu_p"] * np_ + prm["mu_e"] * ne)
    lap = torch.zeros_like(ne)
    for d, hd, dd in ((2, h[0], prm["De"][0]), (1, h[1], prm["De"][1]), (0, h[2], prm["De"][2])):
        n = ne.shape[d]
        if n > 1:
            t = ne.diff(dim=d) * (dd / (hd * hd))
            lap.narrow(d, 0, n - 1).add_(t)
            lap.narrow(d, 1, n - 1).sub_(t)
    return a, np_ - ne - prm["tau_eff"] * lap


def _field(phi, h, pb, pt):
    def centred(lo, hi, d, hd):
        e = torch.cat((lo, phi, hi), dim=d)
        n = phi.shape[d]
        return -(e.narrow(d, 2, n) - e.narrow(d, 0, n)) / (2.0 * hd)

    ex = centred(phi[:, :, :1], phi[:, :, -1:], 2, h[0])
    ey = centred(phi[:, :1], phi[:, -1:], 1, h[1])
    ez = centred(2.0 * pb - phi[:1], 2.0 * pt - phi[-1:], 0, h[2])
    return ex, ey, ez, (ex * ex + ey * ey + ez * ez).sqrt()


def exact(case, seed):
    kind = case["kind"]
    h = (1.0 / case["nx"], 1.0 / case["ny"], 1.0 / case["nz"])
    if kind != "operator" and _cells(case) > 40_000_000:
        return None
    if kind == "step":
        (ne, np_), _, prm = _step_problem(case, seed)
        a, f = _assemble(ne, np_, prm, h)
        phi = _solve(a, f, PB, PT)
        return {"a": a, "f": f, "phi": phi, "E": _field(phi, h, PB, PT)}
    a, f, g = _problem(case, seed)
    if kind == "operator":
        return _apply(f, a, h, PB, PT)
    phi = _solve(a, f, PB, PT)
    if kind in ("solve", "krylov"):
        return phi
    lam = _solve(a, g, 0.0, 0.0)
    out = {"phi": phi, "dLda": _dlda(phi, lam, h, PB, PT)}
    out["dLdf" if kind == "autograd" else "lam"] = lam
    return out
