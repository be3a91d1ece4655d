"""The work that programs have this framework do, as cases that can be timed and checked one by one.

A case names one call (or one short sequence of calls, as a program makes them) of the public entry points in
``paper_2105_06055_amd.binding`` and ``paper_2105_06055_amd.autograd``:

``force``     the internal force density of a displacement field (with the strain energy density where asked)
``verlet``    a multi-step velocity-Verlet call that advances a state in place
``rollout``   a differentiable trajectory: forward, then the gradients of u0, v0 and the micromodulus scale
``solve``     an elastostatic solve by conjugate gradients
``damage``    the damage index of an integrity map

``listed()`` holds one of each kind and direction at the sizes of the repository's own workloads and tests, from the
64 x 64 plate up to the 256^3 block; ``draw()`` gives more of the same ranges.
"""
import math

import numpy as np
import torch

from paper_2105_06055_amd import autograd, binding

F32, F64 = "float32", "float64"


def listed():
    return [
        # the smallest call of the tests and the smoke run: one bond-based force of a 64 x 64 plate
        _case("plate64_force_f64", "force", "bb", F64, 3, nx=64, ny=64, fx=128, fy=128),
        # its trajectory, called a few steps at a time as a program that watches the state does
        _case("plate64_verlet_f32", "verlet", "bb", F32, 3, nx=64, ny=64, fx=128, fy=128, steps=10),
        # the notched glass plate: explicit fracture dynamics with the energy failure rule
        _case("fracture_verlet_f32", "verlet", "bb", F32, 4, nx=1000, ny=400, fx=1024, fy=512, steps=20,
              weight="integrity", dx=1e-4),
        # the same plate on the vertex-centred grid of a refinement study (odd lengths, minimum padding), FP64
        _case("refined_verlet_f64", "verlet", "bb", F64, 6, nx=601, ny=241, fx=640, fy=256, steps=20,
              weight="integrity", dx=1e-3 / 6),
        # force and energy density of a damaged plate, as a post-processing or monitoring call
        _case("damaged_energy_f32", "force", "bb", F32, 3, nx=333, ny=250, fx=384, fy=256, weight="integrity",
              energy=True),
        # inverse problems: gradients of a trajectory on the heterogeneous 512 x 512 plate
        _case("hetero_rollout_f32", "rollout", "bb", F32, 3, nx=512, ny=512, fx=1024, fy=1024, steps=10,
              weight="scale"),
        # large deformations: the nonlinear model on a 3D block
        _case("nonlinear_force_f32", "force", "nbb", F32, 3, nx=128, ny=128, nz=128, fx=256, fy=256, fz=256),
        # the static cube: one FP64 operator application at its size (residual checks, user-written solvers)
        _case("cube128_force_f64", "force", "lps", F64, 3, nx=128, ny=128, nz=128, fx=256, fy=256, fz=256),
        # its solve in the mixed-precision preconditioned form, on a ragged body of a quarter of the size
        _case("cube_solve_mixed", "solve", "lps", F64, 3, nx=81, ny=80, nz=77, fx=96, fy=128, fz=128, mixed=True,
              precond=True),
        # a longer horizon on a ragged body
        _case("horizon4_force_f32", "force", "lps", F32, 4, nx=150, ny=125, nz=100, fx=160, fy=256, fz=128),
        # explicit dynamics of a ragged block in FP64
        _case("block_verlet_f64", "verlet", "lps", F64, 3, nx=201, ny=150, nz=97, fx=256, fy=256, fz=128, steps=10),
        # the headline: explicit dynamics of the 256^3 block with ellipsoidal voids, FP32
        _case("block256_verlet_f32", "verlet", "lps", F32, 3, nx=256, ny=256, nz=256, fx=512, fy=512, fz=512,
              steps=10),
    ]


def _case(name, op, model, dtype, m, nx, ny, fx, fy, nz=1, fz=1, steps=0, weight="none", dx=1e-3, energy=False,
          mixed=False, precond=False):
    case = {"op": op, "model": model, "dtype": dtype, "m": m, "nx": nx, "ny": ny, "nz": nz, "fx": fx, "fy": fy,
            "fz": fz, "dx": dx, "steps": steps, "weight": weight, "energy": energy, "mixed": mixed,
            "precond": precond}
    return dict(case, name=name) if name else case


def _grid(n, m, x=False):
    """Smallest supported box length >= n + m: a power of two, along x also 2 R 2^p with R = 3, 5, 9."""
    need, best = max(16, n + m), 16
    while best < need:
        best *= 2
    if x:
        for r in (3, 5, 9):
            p = 8
            while 2 * r * p < need:
                p *= 2
            best = min(best, 2 * r * p)
    return best


def draw(rng):
    op, model, weight = rng.choice([
        ("force", "bb", "none"), ("force", "bb", "integrity"), ("force", "bb", "scale"), ("force", "lps", "none"),
        ("force", "lps", "none"), ("force", "nbb", "none"), ("verlet", "bb", "integrity"), ("verlet", "bb", "none"),
        ("verlet", "lps", "none"), ("verlet", "lps", "none"), ("rollout", "bb", "scale"), ("solve", "lps", "none"),
        ("solve", "bb", "none"), ("damage", "bb", "integrity")])
    dtype = F64 if op == "solve" else rng.choice([F32, F64])
    dim = 3 if model == "lps" else 2 if weight != "none" else rng.choice([2, 3])
    energy = op == "force" and weight != "none" and rng.random() < 0.5

    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    if dim == 2:
        m = rng.choice([2, 3, 3, 4, 6, 8])
        hi = 320 if op in ("solve", "rollout") else 1000
        n = [size(48, hi), size(40, hi), 1]
    else:
        m = rng.choice([2, 3, 3, 3, 4, 6]) if op != "solve" else rng.choice([2, 3])
        if model == "nbb":
            m = min(m, 3)
        hi = {"solve": 80, "force": 256, "verlet": 256}[op]
        n = [size(24, hi), size(24, hi), size(24, hi)]
        most = {2: 256 ** 3, 3: 256 ** 3, 4: 160 ** 3, 6: 112 ** 3}[m] // (8 if model == "nbb" else 1)
        if dtype == F64 or op == "verlet":
            most //= 2
        while n[0] * n[1] * n[2] > most:
            n[n.index(max(n))] = max(n) * 4 // 5
    odd = rng.random()
    fit = rng.random() < 0.5   # half the programs take minimum padding along x
    if odd < 0.3:
        n[0] += 1 - n[0] % 2
    f = [_grid(n[0], m, x=fit), _grid(n[1], m), _grid(n[2], m) if dim == 3 else 1]
    steps = rng.choice([2, 5, 10]) if op in ("verlet", "rollout") else 0
    mixed = op == "solve" and rng.random() < 0.5
    precond = op == "solve" and rng.random() < 0.5
    return _case(None, op, model, dtype, m, n[0], n[1], f[0], f[1], n[2], f[2], steps, weight, 1e-3, energy, mixed,
                 precond)


# ---------------------------------------------------------------- inputs

_E, _RHO, _RTOL = 72e9, 2440.0, 1e-11


def _nu(c):
    return 0.3 if c["model"] == "lps" else 0.25


def _dim(c):
    return 3 if c["nz"] > 1 else 2


def _body(c):
    return (c["nz"], c["ny"], c["nx"]) if _dim(c) == 3 else (c["ny"], c["nx"])


def _dt(c):
    return 5e-5 * c["dx"]   # a quarter to a third of the stability limit


def _g0(c):
    return 3.8 if c["weight"] == "integrity" else 0.0


def _inputs(c, seed):
    """Masks, fields and loads of a case, on the GPU in FP64 (rounded to the case's type where it has one)."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    dim, body, dx, m = _dim(c), _body(c), c["dx"], c["m"]
    real = torch.float32 if c["dtype"] == F32 else torch.float64

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float64)

    def uniform(*shape):
        return torch.rand(*shape, generator=gen, device="cuda", dtype=torch.float64)

    axes = [torch.arange(n, device="cuda", dtype=torch.float64) + 0.5 for n in body]
    grid = [a.reshape([-1 if k == d else 1 for k in range(dim)]) for d, a in enumerate(axes)]
    chi = torch.ones(body, dtype=torch.bool, device="cuda")
    if dim == 3:
        # voids: axis-aligned ellipsoids inside the body
        at, ax = uniform(8, 3).cpu(), uniform(8, 3).cpu()
        for k in range(8 if min(body) >= 48 else 2):
            r = sum(((grid[d] - body[d] * (0.25 + 0.5 * float(at[k, d]))) /
                     (body[d] * (0.05 + 0.07 * float(ax[k, d])))) ** 2 for d in range(3))
            chi &= r > 1
    free = chi[None].repeat([dim] + [1] * dim).clone()
    if c["op"] == "solve":
        free[:, :3 * m] = False   # a clamped layer three horizons thick
    x = {"chi": chi, "free": free, "u": torch.zeros((dim,) + body, device="cuda", dtype=torch.float64)}
    if c["op"] == "solve":
        x["b"] = (2 * uniform(dim, *body) - 1) * 1e8 * free
        return x
    # a smooth displacement with nodal noise; the nonlinear model takes a tenth of a spacing
    amp = 0.1 * dx if c["model"] == "nbb" else 1e-3 * dx
    ph = (uniform(dim, dim) * 6.28).cpu()
    if c["op"] in ("force", "rollout"):
        for d in range(dim):
            s = sum(torch.sin(6.2831853 * (1 + (k + d) % 2) * grid[k] / body[k] + float(ph[d, k])) for k in range(dim))
            x["u"][d] = amp * (0.2 * s + normal(*body))
    # an impulse on the layer next to the x = 0 face, weak motion elsewhere; plates start under their tractions
    x["v"] = (0.1 if c["weight"] == "integrity" else 0.01) * normal(dim, *body)
    if c["weight"] == "none":
        x["v"][..., :m] += normal(dim, *body[:-1], m)
    x["v"] *= free
    if c["weight"] == "integrity":
        # the notch, a horizon thick, up to half the length, and tractions as body forces on the edge layers
        lam = torch.ones(body, dtype=torch.uint8, device="cuda")
        lam[((grid[0] - body[0] / 2).abs() < m / 2) & (grid[1] < body[1] / 2)] = 0
        if c["op"] != "verlet":
            lam[uniform(*body) < 0.02] = 0
        x["lam"] = lam
        b = torch.zeros_like(x["u"])
        sigma = 4e6 * (1 + 0.2 * float(uniform(1)))
        b[1, -m:], b[1, :m] = sigma / (m * dx), -sigma / (m * dx)
        x["b"] = b
    if c["weight"] == "scale":
        # a micromodulus that varies smoothly by a fifth
        s = sum(torch.sin(6.2831853 * (2 + k) * grid[k] / body[k] + float(ph[0, k])) for k in range(dim))
        x["s"] = torch.sqrt(1 + 0.1 * s)
    if c["op"] == "rollout":
        # cotangents of the final state: a seeded target displacement
        x["ut"] = normal(dim, *body)
        x["vt"] = _dt(c) * normal(dim, *body)
    return {k: (t.to(real).contiguous() if t.dtype == torch.float64 else t) for k, t in x.items()}


def prepare(case, seed):
    c, x = case, _inputs(case, seed)
    dim = _dim(c)
    fft = (c["fz"], c["fy"], c["fx"]) if dim == 3 else (c["fy"], c["fx"])
    plan = binding.Plan(fft, _body(c), c["dx"], c["m"] * c["dx"], model=c["model"], E=_E, nu=_nu(c), rho=_RHO,
                        G0=_g0(c), weight=c["weight"], chiB=x["chi"].cpu().numpy().astype(np.uint8),
                        chiO=x["free"].cpu().numpy().astype(np.uint8),
                        dtype=torch.float32 if c["dtype"] == F32 else torch.float64, mixed=c["mixed"])
    st = {"case": c, "plan": plan, **x}
    if c["op"] == "verlet":
        st["state"] = {"u": x["u"], "v": x["v"], "F": torch.zeros_like(x["u"]), "step": 0}
        if c["weight"] == "integrity":
            st["state"]["lam"] = x["lam"]
            st["state"]["W"] = torch.zeros(_body(c), dtype=x["u"].dtype, device="cuda")
    return st


def run(st):
    c, plan = st["case"], st["plan"]
    if c["op"] == "force":
        w = st.get("lam") if c["weight"] == "integrity" else st.get("s")
        return plan.force(st["u"], weight=w, energy=c["energy"])
    if c["op"] == "verlet":
        s = st["state"]
        plan.verlet(s, _dt(c), c["steps"], b=st.get("b"))
        return {k: t for k, t in s.items() if k != "step"}
    if c["op"] == "rollout":
        u0, v0, s = (st[k].detach().requires_grad_(True) for k in ("u", "v", "s"))
        u, v = autograd.VerletRollout.apply(plan, u0, v0, s, _dt(c), c["steps"], 5)
        gu, gv, gs = torch.autograd.grad([u, v], [u0, v0, s], [st["ut"], st["vt"]])
        return {"u": u.detach(), "v": v.detach(), "gu": gu, "gv": gv, "gs": gs}
    if c["op"] == "solve":
        u, _ = plan.static_solve(st["b"], rtol=_RTOL, mixed=c["mixed"], precond=c["precond"])
        return u
    return plan.damage_index(st["lam"])


# ---------------------------------------------------------------- the work that cannot be left out

def _bonds(c):
    """Offsets o with 0 < |o| <= m, in (x, y, z) order."""
    m, dim = c["m"], _dim(c)
    r = range(-m, m + 1)
    return [(i, j, k) for k in (r if dim == 3 else (0,)) for j in r for i in r if 0 < i * i + j * j + k * k <= m * m]


def work(case):
    c, dim = case, _dim(case)
    n, t = c["nx"] * c["ny"] * c["nz"], 4 if c["dtype"] == F32 else 8
    pairs = len(_bonds(c))
    # multiplications and additions of one force by its bonds: the elongation and the bond force (and the
    # dilatation, for the state-based model); a transform method may do with fewer for long horizons
    points = c["fx"] * c["fy"] * c["fz"]
    fields = {"bb": 2 * dim, "lps": 8, "nbb": 4 * dim + 2 + dim * (dim + 1)}[c["model"]] + (dim if c["weight"] != "none" else 0)
    by_bonds = n * pairs * {"bb": 4 * dim, "lps": 6 * dim + 4, "nbb": 8 * dim}[c["model"]]
    by_transform = 2.5 * fields * points * math.log2(points)
    force = float(min(by_bonds, by_transform))
    wb = {"none": 0, "integrity": 1, "scale": t}[c["weight"]]
    mask = n   # one byte a node
    if c["op"] == "force":
        return {"bytes": 2 * dim * t * n + (t * n if c["energy"] else 0) + wb * n + mask, "flops": force}
    if c["op"] == "verlet":
        # u, v, F read and written once a call, b and the mask read; every step's force
        extra = (2 + 2 * t) * n + dim * t * n if c["weight"] == "integrity" else 0
        return {"bytes": 6 * dim * t * n + extra + mask, "flops": force * c["steps"]}
    if c["op"] == "rollout":
        # the inputs, the cotangents, the results; a force forward, one recomputed and two adjoint ones a step
        return {"bytes": (8 * dim + 2) * t * n + mask, "flops": 5.0 * force * c["steps"]}
    if c["op"] == "solve":
        # the least is a load read and a solution written; iterations grow with the body's length in horizons
        its = 1.5 * max(c["nx"], c["ny"], c["nz"]) / c["m"]
        return {"bytes": 2 * dim * t * n + mask, "flops": force * its}
    return {"bytes": (2 + t) * n, "flops": float(n * pairs)}


# ---------------------------------------------------------------- plain torch in 64 bits

def _constants(c):
    dim, dx, m = _dim(c), c["dx"], c["m"]
    delta, dV = m * dx, dx ** dim
    om = [(o, math.sqrt(sum(q * q for q in o)) * dx) for o in _bonds(c)]
    m0 = sum(r * dV for _, r in om)   # influence 1/r: sum of omega r^2 dV
    moment = math.pi / 4 if dim == 2 else 4 * math.pi / 15
    lame = 3 * _E / 8 if dim == 2 else 2 * _E / 5
    alpha = 2 * lame / (moment * delta ** (dim + 1) / (dim + 1))
    kappa, mu = _E / (3 * (1 - 2 * _nu(c))), _E / (2 * (1 + _nu(c)))
    return delta, dV, om, m0, alpha, kappa, mu


def _pad(f, m, dim):
    return torch.nn.functional.pad(f, [m, m] * dim)


def _at(p, o, body, m):
    """The values of a padded field at x + o."""
    s = [slice(m + q, m + q + n) for q, n in zip(reversed(o[:len(body)]), body)]
    return p[tuple([Ellipsis] + s)]


def _force64(c, u, phi, want_W=False):
    """(L, W) by the sum over bonds; phi is the nodal weight (body mask times integrity or scale)."""
    dim, body, m, dx = _dim(c), _body(c), c["m"], c["dx"]
    delta, dV, om, m0, alpha, kappa, mu = _constants(c)
    up, pp = _pad(u, m, dim), _pad(phi, m, dim)
    L, W = [torch.zeros_like(u[0]) for _ in range(dim)], torch.zeros_like(u[0])
    if c["model"] == "lps":
        mass, theta = torch.zeros_like(phi), torch.zeros_like(phi)
        for o, r in om:
            pn, un = _at(pp, o, body, m), _at(up, o, body, m)
            mass = mass + pn * (r * dV)
            dil = sum((un[d] - u[d]) * (o[d] * dx / r * dV) for d in range(dim) if o[d])
            theta = theta + pn * dil
        theta = torch.where(mass > 0, 3 * phi * theta / mass.clamp_min(1e-300), torch.zeros_like(phi))
        tp = _pad(theta, m, dim)
        ka, kc = (3 * kappa - 5 * mu) / m0, 30 * mu / m0
        for o, r in om:
            pn, un = _at(pp, o, body, m), _at(up, o, body, m)
            el = sum((un[d] - u[d]) * (o[d] * dx) for d in range(dim) if o[d]) * (kc / r ** 3 * dV)
            s = pn * (el + (theta + _at(tp, o, body, m)) * (ka / r * dV))
            for d in range(dim):
                if o[d]:
                    L[d] = L[d] + s * (o[d] * dx)
        return torch.stack(L) * phi, None
    for o, r in om:
        pn = _at(pp, o, body, m)
        eta = _at(up, o, body, m) - u
        el = sum(eta[d] * (o[d] * dx) for d in range(dim) if o[d])
        k = alpha / r ** 3 * dV
        if c["model"] == "nbb":
            s = pn * ((2 * el + (eta * eta).sum(0)) * (k / 2))
            for d in range(dim):
                L[d] = L[d] + s * (o[d] * dx + eta[d])
        else:
            s = pn * el * k
            for d in range(dim):
                if o[d]:
                    L[d] = L[d] + s * (o[d] * dx)
            if want_W:
                W = W + s * el
    return torch.stack(L) * phi, 0.5 * phi * W


def _steps64(c, x, u, v, s=None):
    """The trajectory of `steps` velocity-Verlet steps from (u, v): u, v, F and, with integrity, W."""
    dt, chi, free = _dt(c), x["chi"].double(), x["free"].double()
    lam, b = x.get("lam"), x.get("b")
    fail = _g0(c) / (c["m"] * c["dx"])
    phi = chi if lam is None else chi * lam
    phi = phi if s is None else phi * s
    b = 0.0 if b is None else b.double()
    L, W = _force64(c, u, phi, lam is not None)
    F = L + b
    for _ in range(c["steps"]):
        u = free * (u + dt * v + dt * dt / (2 * _RHO) * F)
        if lam is not None:
            phi = phi * (W <= fail)
        L, W = _force64(c, u, phi, lam is not None)
        new = L + b
        v = free * (v + dt / (2 * _RHO) * (F + new))
        F = new
    return u, v, F, W


def _solve64(c, x):
    """Conjugate gradients on the free components, the operator applied by torch's transforms of the whole box."""
    dim, body = 3 if c["nz"] > 1 else 2, _body(c)
    delta, dV, om, m0, alpha, kappa, mu = _constants(c)
    lps, dx = c["model"] == "lps", c["dx"]
    box = [n + c["m"] for n in body]
    K, A = {}, [torch.zeros(box, device="cuda", dtype=torch.float64) for _ in range(dim)]
    M = torch.zeros(box, device="cuda", dtype=torch.float64)
    for i in range(dim):
        for j in range(i, dim):
            K[i, j] = torch.zeros(box, device="cuda", dtype=torch.float64)
    for o, r in om:
        at = tuple((-q) % n for q, n in zip(reversed(o[:dim]), box))
        for i, j in K:
            K[i, j][at] = (30 * mu / m0 if lps else alpha) / r ** 3 * o[i] * o[j] * dx * dx * dV
        for i in range(dim):
            A[i][at] = o[i] * dx / r * dV
        M[at] = r * dV
    hat = torch.fft.rfftn
    K, A, M = {k: hat(v) for k, v in K.items()}, [hat(a) for a in A], hat(M)
    crop = tuple(slice(0, n) for n in body)
    chi, free = x["chi"].double(), x["free"].double()

    def spec(f):
        return torch.fft.rfftn(f, s=box)

    def back(f):
        return torch.fft.irfftn(f, s=box)[crop]

    pair = lambda i, j: K[min(i, j), max(i, j)]  # noqa: E731
    ch = spec(chi)
    G = {k: back(K[k] * ch) for k in K}
    g, mass = [back(a * ch) for a in A], back(M * ch)
    ka = (3 * kappa - 5 * mu) / m0

    def apply(u):
        U = [spec(chi * u[d]) for d in range(dim)]
        S = [sum(pair(i, j) * U[j] for j in range(dim)) for i in range(dim)]
        if lps:
            th = back(sum(A[d] * U[d] for d in range(dim))) - sum(g[d] * u[d] for d in range(dim))
            th = torch.where(mass > 1e-30, 3 * chi * th / mass.clamp_min(1e-30), torch.zeros_like(th))
            T = spec(th)
            S = [S[i] + ka * A[i] * T for i in range(dim)]
        out = [back(S[i]) - sum(G[min(i, j), max(i, j)] * u[j] for j in range(dim)) for i in range(dim)]
        if lps:
            out = [out[i] + ka * th * g[i] for i in range(dim)]
        return -torch.stack(out) * chi * free

    u, r = torch.zeros_like(x["b"]), x["b"] * free
    p, rr = r.clone(), (r * r).sum()
    stop = rr * 1e-26
    for k in range(3000):
        q = apply(p)
        a = rr / (p * q).sum()
        u, r = u + a * p, r - a * q
        new = (r * r).sum()
        if k % 16 == 15 and bool(new < stop):
            break
        p, rr = r + (new / rr) * p, new
    return u


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    if c["op"] == "solve":
        return _solve64(c, x)
    chi = x["chi"].double()
    if c["op"] == "damage":
        lam, pad, cnt, fam = chi * x["lam"], c["m"], 0.0, 0.0
        lp, cp = _pad(lam, pad, 2), _pad(chi, pad, 2)
        for o, _ in _constants(c)[2]:
            cnt, fam = cnt + _at(lp, o, _body(c), pad), fam + _at(cp, o, _body(c), pad)
        return torch.where(chi > 0, 1 - lam * (cnt + lam) / (chi + fam).clamp_min(1), torch.zeros_like(chi))
    u = x["u"].double()
    if c["op"] == "force":
        phi = chi * x["lam"] if c["weight"] == "integrity" else chi * x["s"].double() if c["weight"] == "scale" else chi
        L, W = _force64(c, u, phi, c["energy"])
        return (L, W) if c["energy"] else L
    if c["op"] == "verlet":
        u, v, F, W = _steps64(c, x, u, x["v"].double())
        out = {"u": u, "v": v, "F": F}
        return dict(out, lam=None, W=W) if c["weight"] == "integrity" else out
    u0, v0, s = (x[k].double().requires_grad_(True) for k in ("u", "v", "s"))
    u, v, _, _ = _steps64(c, x, u0, v0, s)
    gu, gv, gs = torch.autograd.grad([u, v], [u0, v0, s], [x["ut"].double(), x["vt"].double()])
    return {"u": u.detach(), "v": v.detach(), "gu": gu, "gv": gv, "gs": gs}
