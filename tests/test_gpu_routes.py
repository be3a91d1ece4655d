"""Which kernels a plate at eight spacings runs (the rule by measured costs in
dir_plan)."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

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
