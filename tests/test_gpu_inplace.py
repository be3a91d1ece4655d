"""Calls whose results go to the buffers of their inputs: the force in place,
the adjoints into their cotangent, displacement or weight.  The results are
those of the same call with buffers of its own, bit for bit: the arithmetic is
the same and only the addresses differ.  Bodies of many blocks, so that a
block's neighbours have inputs that another block's results replace."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_06055_amd import workloads as wl

pytestmark = pytest.mark.gpu

DT = [torch.float64, torch.float32]


def _dev(a, dtype):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _plan(body, dtype, model="bb", weight="none"):
    from paper_2105_06055_amd import binding
    return binding.Plan(tuple(wl._grid_len(n, 3) for n in body), body, 1e-3, 3e-3, model=model, E=70e9, nu=0.3,
                        rho=2440.0, chiB=wl.random_mask(body, 71), weight=weight, dtype=dtype)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("mode", ["auto", "yfft"])
@pytest.mark.parametrize("model,weight,body", [("lps", "none", (41, 50, 67)), ("bb", "none", (41, 50, 67)),
                                               ("nbb", "none", (41, 50, 67)), ("bb", "none", (150, 201)),
                                               ("nbb", "none", (150, 201)), ("bb", "integrity", (150, 201)),
                                               ("bb", "scale", (150, 201))])
def test_force_in_place(dtype, mode, model, weight, body):
    plan = _plan(body, dtype, model, weight)
    plan.set_lastaxis(mode)
    rng = np.random.default_rng(72)
    u = _dev(rng.normal(0, 1e-6, (len(body),) + body), dtype)
    wt = None
    if weight == "integrity":
        wt = _dev(rng.random(body) > 0.2, torch.uint8)
    if weight == "scale":
        wt = _dev(rng.uniform(0.8, 1.2, body), dtype)
    ref = plan.force(u, weight=wt)
    x = u.clone()
    plan.force(x, weight=wt, out=x)
    assert torch.equal(x, ref)
    if weight == "scale":   # L over the weight: s is the first component of the result's buffer
        x = torch.stack([wt, wt])
        plan.force(u, weight=x[0], out=x)
        assert torch.equal(x, ref)
    plan.close()


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("model,body", [("lps", (41, 50, 67)), ("bb", (41, 50, 67)), ("bb", (150, 201))])
def test_force_adjoint_in_place(dtype, model, body):
    from paper_2105_06055_amd import binding
    plan = _plan(body, dtype, model)
    rng = np.random.default_rng(73)
    g = _dev(rng.normal(0, 1.0, (len(body),) + body), dtype)
    ref = plan.force_adjoint(g, g)
    x = g.clone()
    binding._check(binding.lib().pd_force_adjoint(plan._h, None, None, C.c_void_p(x.data_ptr()),
                                                  C.c_void_p(x.data_ptr()), None, binding._stream()), "adjoint")
    assert torch.equal(x, ref)
    plan.close()


@pytest.mark.parametrize("dtype", DT)
def test_weight_adjoint_in_place(dtype):
    """u_bar over the cotangent or over u, weight_bar over the weight."""
    from paper_2105_06055_amd import binding
    body = (150, 201)
    plan = _plan(body, dtype, "bb", "scale")
    rng = np.random.default_rng(74)
    u, g = (_dev(rng.normal(0, 1e-6, (2,) + body), dtype) for _ in range(2))
    s = _dev(rng.uniform(0.8, 1.2, body), dtype)
    ub, sb = plan.force_adjoint(u, g, weight=s, want_weight_bar=True)
    for over in ("g", "u"):
        x = {"u": u.clone(), "g": g.clone(), "s": s.clone()}
        at = {k: C.c_void_p(t.data_ptr()) for k, t in x.items()}
        binding._check(binding.lib().pd_force_adjoint(plan._h, at["u"], at["s"], at["g"], at[over], at["s"],
                                                      binding._stream()), "adjoint")
        assert torch.equal(x[over], ub) and torch.equal(x["s"], sb), over
    plan.close()


@pytest.mark.parametrize("dtype", DT)
def test_verlet_adjoint_over_states(dtype):
    """The cotangents are the states themselves (a loss of |u_n|^2 / 2): u_bar
    over u_n or u_np1, v_bar over u_n."""
    body, dt = (150, 201), 2e-8
    plan = _plan(body, dtype, "bb", "scale")
    rng = np.random.default_rng(75)
    un, up = (_dev(rng.normal(0, 1e-6, (2,) + body), dtype) for _ in range(2))
    s = _dev(rng.uniform(0.8, 1.2, body), dtype)

    def run(alias):
        x = {"un": un.clone(), "up": up.clone()}
        ub = x[alias["ub"]] if "ub" in alias else un.clone() if alias["like"][0] == "un" else up.clone()
        vb = x[alias["vb"]] if "vb" in alias else un.clone()
        sb, bb = torch.zeros_like(s), torch.zeros_like(un)
        plan.verlet_adjoint(x["un"], x["up"], ub, vb, dt, s=s, s_bar=sb, b_bar=bb)
        return ub, vb, sb, bb

    for alias in ({"ub": "un"}, {"ub": "up"}, {"ub": "up", "vb": "un"}):
        ref = run({"like": (alias["ub"],)})
        for a, b in zip(run(alias), ref):
            assert torch.equal(a, b), alias
    plan.close()
