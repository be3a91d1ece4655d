"""Which kernels a plate at eight spacings runs (the rule by measured costs in
dir_plan), and the unweighted calls at the radii on both sides of the rules."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_06055_amd import workloads as wl

import parity

pytestmark = pytest.mark.gpu


def _dev(a, dtype=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


class _Pass(C.Structure):
    _fields_ = [("name", C.c_char * 32), ("launches", C.c_int64), ("total_ms", C.c_double), ("bytes", C.c_double)]


def _passes(plan, call):
    from paper_2105_06055_amd import binding
    L = binding.lib()
    L.pd_profile_enable.argtypes = [C.c_void_p, C.c_int]
    L.pd_profile_read.argtypes = [C.c_void_p, C.POINTER(_Pass), C.c_int, C.POINTER(C.c_int)]
    binding._check(L.pd_profile_enable(plan._h, 1), "pd_profile_enable")
    call()
    buf, n = (_Pass * 32)(), C.c_int()
    binding._check(L.pd_profile_read(plan._h, buf, 32, C.byref(n)), "pd_profile_read")
    binding._check(L.pd_profile_enable(plan._h, 0), "pd_profile_enable")
    return {buf[i].name.decode() for i in range(n.value)}


@pytest.mark.parametrize("m", [7, 8])
@pytest.mark.parametrize("dtype,body,fft,direct", [
    (torch.float64, (1000, 1000), (1024, 1024), False), (torch.float64, (700, 700), (1024, 1024), True),
    (torch.float64, (900, 1400), (1024, 2048), True), (torch.float64, (900, 1900), (1024, 2048), False),
    (torch.float32, (1000, 1000), (1024, 1024), True), (torch.float32, (1010, 2030), (1024, 2048), False)])
def test_plate_of_eight_spacings(dtype, body, fft, direct, m):
    """Large plates that fill their grid take the transforms, the others and
    every call with the energy density the bond sums; the forces agree (FP64
    1e-12, FP32 1e-5 of the largest value: both are within a few roundings of
    the sums)."""
    from paper_2105_06055_amd import binding
    plan = binding.Plan(fft, body, 1e-3, m * 1e-3, E=72e9, dtype=dtype)
    u = _dev(np.random.default_rng(94).normal(0, 1e-6, (2,) + body), dtype)
    out = {}
    names = _passes(plan, lambda: out.update(L=plan.force(u)))
    assert ("dir2_m8" in names) == direct and ("xfwd_2" in names) != direct, names
    names = _passes(plan, lambda: out.update(E=plan.force(u, energy=True)))
    assert names == {"dir2_m8"}, names
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    assert float((out["L"] - out["E"][0]).abs().max() / out["L"].abs().max()) <= tol
    plan.close()


@pytest.mark.parametrize("m", [3, 5, 6, 8])
def test_unweighted_plate_adjoint_and_energies(orc, m):
    """The reverse steps of an unweighted plate (one kernel per half up to five
    spacings, operator calls beyond) and a step's energies without W."""
    from paper_2105_06055_amd import binding
    body, dx, rho, dt, nsteps = (33, 41), 1e-3, 2440.0, 2e-8, 3
    chi = wl.random_mask(body, 95)
    omega = np.stack([chi] * 2)
    omega[:, :2] = 0
    rng = np.random.default_rng(96)
    plan = binding.Plan(tuple(wl._grid_len(n, m) for n in body), body, dx, m * dx, E=72e9, rho=rho, chiB=chi,
                        chiO=omega, dtype=torch.float64)
    g, al = orc.geom(body, dx, m * dx), orc.bb_alpha(2, 72e9, m * dx)
    u, v = rng.normal(0, 1e-6, (2,) + body) * omega, rng.normal(0, 1.0, (2,) + body) * omega
    gu, gv = rng.normal(0, 1.0, (2,) + body), rng.normal(0, 1e-8, (2,) + body)
    st = {"u": _dev(u), "v": _dev(v), "F": torch.zeros((2,) + body, dtype=torch.float64, device="cuda"), "step": 0}
    us = [st["u"].clone()]
    en = []
    for _ in range(nsteps):
        en.append(plan.verlet(st, dt, 1, energy=True)[0])
        us.append(st["u"].clone())
    ub, vb = _dev(gu), _dev(gv)
    for k in range(nsteps - 1, -1, -1):
        plan.verlet_adjoint(us[k], us[k + 1], ub, vb, dt)
    uo, vo, _ = orc.verlet_adjoint(g, al, rho, omega, chi.astype(float), np.zeros((2,) + body), u, v, dt, nsteps, gu,
                                   gv)
    assert parity.rel_max(ub.cpu().numpy(), uo) <= 1e-11 and parity.rel_max(vb.cpu().numpy(), vo) <= 1e-11
    # the energies of the last step from the oracle's force of its state
    un, vn = (st[k].cpu().numpy() for k in ("u", "v"))
    Lo, dV = orc.bb_force(g, al, chi.astype(float), un), dx * dx
    ke, pe, sh = 0.5 * rho * np.sum(vn ** 2) * dV, -0.5 * np.sum(un * Lo) * dV, np.sum((omega * Lo) ** 2) * dV
    ref = np.array([ke, pe, 0.0, ke + pe - dt * dt / (8 * rho) * sh])
    assert np.max(np.abs(np.array(en[-1]) - ref)) <= 1e-11 * np.max(np.abs(ref))
    plan.close()
