"""Direct horizon sums (csrc/pd_direct.hpp, pd_direct2.hpp) against the FP64
oracle where they can go wrong: edges of the 32 x 8 tiles (and the 32 x 16
pair tiles of the FP64 dilatation, odd rows), chunks along z of one plane and
more, bodies smaller than a tile, every compiled radius, horizons between
spacings (kernel values beyond them are zero), the steps' forms (first, inner
and last of a call; exact steps; prescribed displacement, load), and plans
that do not qualify (unequal spacings), which keep the transform path.

Bars: those of tests/parity.py for forces.  A Verlet step multiplies the force
error by dt^2 / rho at most, so states keep the FP64 force bar and take 1e-5
in FP32 (the FP32 force bar times dt^2 lambda_max / rho <= 4, with room for
the rounding of u + dt v).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_06055_amd import workloads as wl

import parity

pytestmark = pytest.mark.gpu

DT = [torch.float64, torch.float32]


def _dev(a, dtype):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _fft(body, m):
    return tuple(wl._grid_len(n, int(np.ceil(m))) for n in body)


def _rel(x, ref):
    return float(np.max(np.abs(x - ref)) / np.max(np.abs(ref)))


# (z, y, x): one node more and less than a tile, a row of one node, odd and
# even rows, planes fewer than the horizon
BODIES3 = [((5, 9, 33), 3.0), ((21, 17, 32), 3.0), ((2, 8, 31), 2.0), ((40, 7, 1), 2.0), ((13, 16, 65), 4.0),
           ((9, 24, 30), 2.3)]


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("model", ["lps", "bb", "nbb"])
@pytest.mark.parametrize("body,m", BODIES3)
def test_3d_force(orc, dtype, model, body, m):
    from paper_2105_06055_amd import binding
    dx, rho = 1e-3, 2700.0
    chi = wl.random_mask(body, 11)
    plan = binding.Plan(_fft(body, m), body, dx, m * dx, model=model, E=70e9, nu=0.3, rho=rho, chiB=chi, dtype=dtype)
    u = wl.random_field((3,) + body, 12, 1e-6)
    L = plan.force(_dev(u, dtype)).cpu().numpy()
    g = orc.geom(body, dx, m * dx)
    al = orc.bb_alpha(3, 70e9, m * dx)
    if model == "lps":
        Lo, _ = orc.lps_force(g, 70e9, 0.3, chi.astype(float), u)
    else:
        Lo = (orc.bb_force if model == "bb" else orc.nbb_force)(g, al, chi.astype(float), u)
    parity.check_force(L, Lo, u, plan, rho, dtype == torch.float64, f"{model} {body} m={m}")
    plan.close()


@pytest.mark.parametrize("dtype", DT)
def test_3d_steps(orc, dtype):
    """One call of four steps (first, inner, last), the same as exact steps and
    as single calls, with a load and a prescribed displacement, against the
    oracle; exact steps equal single calls bit for bit."""
    from paper_2105_06055_amd import binding
    body, m, dx, rho, dt, n = (19, 10, 35), 3, 1e-3, 2700.0, 5e-8, 4
    chi = wl.random_mask(body, 21)
    omega = np.stack([chi] * 3)
    omega[:, :, :2] = 0
    rng = np.random.default_rng(22)
    u, v = rng.normal(0, 1e-6, (3,) + body), rng.normal(0, 1.0, (3,) + body) * omega
    b, w = rng.normal(0, 1e9, (3,) + body), rng.normal(0, 1e-6, (3,) + body)
    mdl = orc.model("lps", E=70e9, nu=0.3, rho=rho)
    o = orc.verlet(orc.geom(body, dx, m * dx), mdl, chi, omega, u, v, dt, n, b=b, w=w)
    plan = binding.Plan(_fft(body, m), body, dx, m * dx, model="lps", E=70e9, nu=0.3, rho=rho, chiB=chi, chiO=omega,
                        dtype=dtype)

    def run(calls, **kw):
        st = {"u": _dev(u, dtype), "v": _dev(v, dtype), "F": _dev(0 * u, dtype), "step": 0}
        for k in calls:
            plan.verlet(st, dt, k, b=_dev(b, dtype), w=_dev(w, dtype), **kw)
        return st

    states = {"call": run([n]), "exact": run([n], exact_steps=True), "single": run([1] * n),
              "energy": run([n], energy=True), "unchecked": run([n], status=False)}
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    for name, st in states.items():
        for k in ("u", "v", "F"):
            assert _rel(st[k].cpu().numpy(), o[k]) <= tol, (name, k)
    for k in ("u", "v", "F"):
        assert torch.equal(states["exact"][k], states["single"][k]), k
    plan.close()


# (y, x)
BODIES2 = [((9, 33), 3.0), ((8, 32), 2.0), ((41, 1), 2.5), ((17, 70), 4.0), ((30, 45), 5.0), ((23, 64), 6.0),
           ((33, 50), 7.0), ((25, 31), 8.0)]


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("body,m", BODIES2)
def test_2d_force_energy_adjoint_damage(orc, dtype, body, m):
    from paper_2105_06055_amd import binding
    dx, rho = 1e-3, 2440.0
    chi = wl.random_mask(body, 31)
    rng = np.random.default_rng(32)
    u, gb = rng.normal(0, 1e-6, (2,) + body), rng.normal(0, 1.0, (2,) + body)
    lam = (rng.random(body) > 0.2).astype(np.uint8)
    s = rng.uniform(0.8, 1.2, body)
    g, al = orc.geom(body, dx, m * dx), orc.bb_alpha(2, 72e9, m * dx)
    f64 = dtype == torch.float64
    tol = 1e-12 if f64 else 1e-4

    def plan_of(weight, model="bb"):
        return binding.Plan(_fft(body, m), body, dx, m * dx, model=model, E=72e9, rho=rho, G0=3.8, weight=weight,
                            chiB=chi, dtype=dtype)

    for weight, phi, arg in (("none", chi.astype(float), None), ("integrity", chi * lam.astype(float), lam),
                             ("scale", chi * s, s)):
        plan = plan_of(weight)
        wt = None if arg is None else _dev(arg, torch.uint8 if weight == "integrity" else dtype)
        L, W = plan.force(_dev(u, dtype), weight=wt, energy=True)
        parity.check_force(L.cpu().numpy(), orc.bb_force(g, al, phi, u), u, plan, rho, f64, f"{weight} {body} m={m}")
        assert _rel(W.cpu().numpy(), orc.bb_energy(g, al, phi, u)) <= tol, weight
        if weight == "scale":
            ub, sb = plan.force_adjoint(_dev(u, dtype), _dev(gb, dtype), weight=wt, want_weight_bar=True)
            uo, po = orc.bb_force_adjoint(g, al, phi, u, gb)
            assert _rel(ub.cpu().numpy(), uo) <= tol and _rel(sb.cpu().numpy(), po * chi) <= tol
        if weight == "integrity":
            d, _ = orc.damage_index(g, chi, lam)
            # a quotient of counts, rounded once to the plan's type
            assert np.array_equal(plan.damage_index(wt).cpu().numpy(), d.astype(np.float64 if f64 else np.float32))
        plan.close()
    plan = plan_of("none", "nbb")
    L = plan.force(_dev(u, dtype)).cpu().numpy()
    parity.check_force(L, orc.nbb_force(g, al, chi.astype(float), u), u, plan, rho, f64, f"nbb {body} m={m}")
    plan.close()


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("dx,m", [((1e-3, 1e-3, 0.5e-3), 3), ((1e-3, 1e-3, 0.8e-3), 2)])
def test_unequal_spacings_keep_the_transforms(orc, dtype, dx, m):
    """Plans with another spacing along x do not qualify for the direct sums:
    x transform and (y, z) correlation (spacings in (z, y, x) order)."""
    from paper_2105_06055_amd import binding
    body, rho, delta = (14, 15, 20), 2700.0, m * 1e-3
    chi = wl.random_mask(body, 41)
    u = wl.random_field((3,) + body, 42, 1e-6)
    g = orc.geom(body, list(reversed(dx)), delta)
    for model in ("lps", "bb"):
        plan = binding.Plan((32, 32, 64), body, dx, delta, model=model, E=70e9, nu=0.3, rho=rho, chiB=chi, dtype=dtype)
        if model == "lps":
            Lo, _ = orc.lps_force(g, 70e9, 0.3, chi.astype(float), u)
        else:
            Lo = orc.bb_force(g, orc.bb_alpha(3, 70e9, delta), chi.astype(float), u)
        for mode in ("auto", "yfft"):
            plan.set_lastaxis(mode)
            L = plan.force(_dev(u, dtype)).cpu().numpy()
            parity.check_force(L, Lo, u, plan, rho, dtype == torch.float64, f"{model} {dx} {mode}")
        plan.close()


def test_static_solve_component_blocks(orc):
    """The preconditioned solve on a ragged body with a mixed-radix x grid (a
    component per block in its x passes): the oracle's residual of the result."""
    from paper_2105_06055_amd import binding
    body, m, dx, rtol = (11, 18, 21), 3, 1e-3, 1e-10
    w = wl.cube_void_static(nb=12, nfft=16)
    chi = wl.random_mask(body, 51)
    omega = np.stack([chi] * 3)
    omega[:, :3] = 0
    b = np.random.default_rng(52).uniform(-1, 1, (3,) + body) * 1e8 * omega
    g = orc.geom(body, dx, m * dx)
    for mixed in (False, True):
        plan = binding.Plan((16, 32, 48), body, dx, m * dx, model="lps", E=w.E, nu=w.nu, chiB=chi, chiO=omega,
                            dtype=torch.float64, mixed=mixed)
        u, info = plan.static_solve(_dev(b, torch.float64), rtol=rtol, mixed=mixed, precond=True)
        Lo, _ = orc.lps_force(g, w.E, w.nu, chi.astype(float), u.cpu().numpy())
        r = (Lo + b) * omega
        # the library's own FP64 residual is <= rtol; the oracle's differs by the rounding of L
        assert np.linalg.norm(r) / np.linalg.norm(b) <= 2 * rtol, mixed
        plan.close()


# (z, y, x) or (y, x): last-axis lines of 64 and 128 points, three and four taps
LINES = [((50, 13, 18), 2, (64, 16, 32)), ((100, 10, 17), 3, (128, 16, 32)), ((58, 12, 20), 3, (64, 16, 32)),
         ((110, 9, 12), 2, (128, 16, 16)), ((55, 37), 2, (64, 64)), ((110, 30), 3, (128, 64))]


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("body,m,grid", LINES)
def test_preconditioner_short_lines(orc, body, m, grid, mixed):
    """Preconditioned solves whose last axis has 64 or 128 points: the oracle's
    residual, and in FP64 the iteration count of the runtime-length kernel with
    the same operator kernels, those of the transform modes (another rounding
    of the preconditioner may move the end by an iteration or two; another
    operator moves the slender bodies' 260 iterations by up to 15)."""
    from paper_2105_06055_amd import binding
    dx, rtol, D = 1e-3, 1e-10, len(body)
    chi = np.ones(body, dtype=np.uint8)
    omega = np.stack([chi] * D)
    omega[:, :3] = 0
    b = np.random.default_rng(61).uniform(-1, 1, (D,) + body) * 1e8 * omega
    its = {}
    # (mixed on the default path alone: the FP32 operator of the transform modes
    # does not carry the slender bodies to 1e-10, with either kernel)
    for mode in ("auto",) if mixed else ("auto", "fft", "fft_generic"):
        plan = binding.Plan(grid, body, dx, m * dx, model="lps" if D == 3 else "bb", E=60e9, nu=0.3, chiB=chi,
                            chiO=omega, dtype=torch.float64, mixed=mixed)
        plan.set_lastaxis(mode)
        u, info = plan.static_solve(_dev(b, torch.float64), rtol=rtol, mixed=mixed, precond=True)
        its[mode] = info["iters_fp64"]
        g = orc.geom(body, dx, m * dx)
        un = u.cpu().numpy()
        if D == 3:
            Lo, _ = orc.lps_force(g, 60e9, 0.3, chi.astype(float), un)
        else:
            Lo = orc.bb_force(g, orc.bb_alpha(2, 60e9, m * dx), chi.astype(float), un)
        # the library's own FP64 residual is <= rtol; the oracle's differs by the rounding of L
        assert np.linalg.norm((Lo + b) * omega) / np.linalg.norm(b) <= 2 * rtol, mode
        plan.close()
    if not mixed:
        assert abs(its["fft"] - its["fft_generic"]) <= 2, its
