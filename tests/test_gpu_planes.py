"""The 3D direct sums with several planes per block: accumulators carried over
the planes, the LDS ring reused (chunks longer than the horizon), chunks longer
than the accumulators' reach (2 m) and a shorter last one, at every radius;
force, the forms of a Verlet step, energies and the solver's operator, against
the oracle.  (The rule takes one plane per block for bodies of this size.)

Bars as in test_gpu_direct: forces those of tests/parity.py, states 1e-12 in
FP64 and 1e-5 in FP32 of a field's largest value; energies 1e-11 and 1e-5 of the
largest (sums of squares and products of such fields)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_06055_amd import workloads as wl

import parity

pytestmark = pytest.mark.gpu

DT = [torch.float64, torch.float32]
# (m, planes): one, fewer than the horizon, longer than 2 m with a ragged last chunk, the whole body
CASES = [(2, 1), (2, 2), (2, 5), (2, 23), (3, 1), (3, 2), (3, 8), (3, 23), (4, 1), (4, 3), (4, 9), (4, 23)]


def _dev(a, dtype):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _plan(body, m, model, chi, omega, dtype, **kw):
    from paper_2105_06055_amd import binding
    return binding.Plan(tuple(wl._grid_len(n, m) for n in body), body, 1e-3, m * 1e-3, model=model, E=70e9, nu=0.3,
                        rho=2700.0, chiB=chi, chiO=omega, dtype=dtype, **kw)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("model", ["lps", "bb"])
@pytest.mark.parametrize("m,planes", CASES)
def test_force_and_steps(orc, dtype, model, m, planes):
    # odd rows, where the FP64 dilatation's pairs end with one node
    body, dx, rho, dt, n = (23, 10, 35), 1e-3, 2700.0, 5e-8, 4
    chi = wl.random_mask(body, 101)
    omega = np.stack([chi] * 3)
    omega[:, :, :2] = 0
    rng = np.random.default_rng(102)
    u, v = rng.normal(0, 1e-6, (3,) + body), rng.normal(0, 1.0, (3,) + body) * omega
    b, w = rng.normal(0, 1e9, (3,) + body) * chi, rng.normal(0, 1e-6, (3,) + body)
    plan = _plan(body, m, model, chi, omega, dtype)
    plan.set_planes(planes)
    g, al, f64 = orc.geom(body, dx, m * dx), orc.bb_alpha(3, 70e9, m * dx), dtype == torch.float64

    def force(x):
        return orc.lps_force(g, 70e9, 0.3, chi.astype(float), x)[0] if model == "lps" else \
            orc.bb_force(g, al, chi.astype(float), x)

    L = plan.force(_dev(u, dtype)).cpu().numpy()
    parity.check_force(L, force(u), u, plan, rho, f64, f"{model} m={m} planes={planes}")
    mdl = orc.model(model, E=70e9, nu=0.3, rho=rho, alpha=al)
    tol = 1e-12 if f64 else 1e-5

    def run(**kw):
        st = {"u": _dev(u, dtype), "v": _dev(v, dtype), "F": _dev(0 * u, dtype), "step": 0}
        return st, plan.verlet(st, dt, n, b=_dev(b, dtype), **kw)

    for wv in (None, w):
        o = orc.verlet(g, mdl, chi, omega, u, v, dt, n, b=b, w=wv, energy=True)
        ww = None if wv is None else _dev(wv, dtype)
        for kw in ({}, {"exact_steps": True}, {"energy": True}):
            st, en = run(w=ww, **kw)
            for k in ("u", "v", "F"):
                e = parity.rel_max(st[k].cpu().numpy(), o[k])
                assert e <= tol, (kw, k, e)
        assert np.max(np.abs(en - o["energy"])) <= (1e-11 if f64 else 1e-5) * np.max(np.abs(o["energy"]))
    plan.close()


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("m,planes", [(2, 5), (3, 8), (3, 2), (4, 9)])
def test_solve(orc, m, planes, mixed):
    body, dx, rtol = (23, 10, 19), 1e-3, 1e-10
    chi = np.ones(body, dtype=np.uint8)
    chi[9:13, 4:6, 7:11] = 0
    omega = np.stack([chi] * 3)
    omega[:, :3] = 0
    b = np.random.default_rng(103).uniform(-1, 1, (3,) + body) * 1e8 * omega
    plan = _plan(body, m, "lps", chi, omega, torch.float64, mixed=mixed)
    plan.set_planes(planes)
    u, info = plan.static_solve(_dev(b, torch.float64), rtol=rtol, mixed=mixed)
    Lo, _ = orc.lps_force(orc.geom(body, dx, m * dx), 70e9, 0.3, chi.astype(float), u.cpu().numpy())
    # the library's own FP64 residual is <= rtol; the oracle's differs by the rounding of L
    assert np.linalg.norm((Lo + b) * omega) / np.linalg.norm(b) <= 2 * rtol
    plan.close()
