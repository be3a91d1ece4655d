"""FP32 forces of the direct bond sums against FP64 references: the L2 error over
the field relative to the field, in units of u = 2^-24.

The terms of a bond go through about six roundings (the difference of the
displacements, the elongation, its product with the kernel value and the
weight, the sums), each of rms ~0.4 u of the term, and the bonds' errors add up
as the bonds themselves do, so a force is off by about u; 1.5 u leaves room for
the sums.  A factor of all bonds that is rounded (the spacing: off by 0.98 u
here, once in the elongation and once in the direction) would add its whole
error to every force."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_06055_amd import workloads as wl

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -24
DX = 2.0 ** -10 * (1 + 0.98 * ULP)   # rounds to 2^-10 in FP32


def _field(body, amp, seed):
    """A smooth field with nodal noise, as the oracle and the GPU both hold it."""
    rng = np.random.default_rng(seed)
    g = np.meshgrid(*[(np.arange(n) + 0.5) / n for n in body], indexing="ij")
    u = np.stack([sum(np.sin(2 * np.pi * (1 + (k + d) % 2) * x + rng.uniform(0, 6)) for k, x in enumerate(g))
                  for d in range(len(body))])
    return (amp * (0.2 * u + rng.standard_normal(u.shape))).astype(np.float32)


def _error(L, Lo):
    return float(np.linalg.norm(L.double().cpu().numpy() - Lo) / np.linalg.norm(Lo)) / ULP


@pytest.mark.parametrize("body,m", [((90, 131), 2), ((90, 131), 3), ((90, 131), 4), ((90, 131), 6), ((90, 131), 8),
                                    ((25, 34, 43), 2), ((25, 34, 43), 3)])
def test_nonlinear_force_fp32(orc, body, m):
    from paper_2105_06055_amd import binding
    u = _field(body, 0.1 * DX, 91)
    plan = binding.Plan(tuple(wl._grid_len(n, m) for n in body), body, DX, m * DX, model="nbb", E=72e9,
                        dtype=torch.float32)
    Lo = orc.nbb_force(orc.geom(body, DX, m * DX), orc.bb_alpha(len(body), 72e9, m * DX), np.ones(body),
                       u.astype(np.float64))
    e = _error(plan.force(torch.tensor(u, device="cuda")), Lo)
    print(f"nonlinear {body} m={m}: {e:.2f} u", flush=True)
    assert e <= 1.5, e
    plan.close()


@pytest.mark.parametrize("m", [2, 3, 4, 6, 8])
def test_plate_force_fp32_against_transforms(orc, m):
    """The unweighted plate: no less accurate than the transform chain of the
    same plan (a tenth for two sets of roundings on 23,600 values)."""
    from paper_2105_06055_amd import binding
    body = (90, 131)
    u = _field(body, 1e-3 * DX, 92)
    plan = binding.Plan(tuple(wl._grid_len(n, m) for n in body), body, DX, m * DX, E=72e9, dtype=torch.float32)
    Lo = orc.bb_force(orc.geom(body, DX, m * DX), orc.bb_alpha(2, 72e9, m * DX), np.ones(body), u.astype(np.float64))
    e = {}
    for mode in ("auto", "yfft"):
        plan.set_lastaxis(mode)
        e[mode] = _error(plan.force(torch.tensor(u, device="cuda")), Lo)
    print(f"plate m={m}: direct {e['auto']:.2f} u, transforms {e['yfft']:.2f} u", flush=True)
    assert e["auto"] <= 1.1 * e["yfft"], e
    plan.close()


@pytest.mark.parametrize("body,m", [((31, 33), 3), ((31, 33), 5), ((31, 33), 8)])
def test_kernel_values_fp64(body, m):
    """The FP64 force of a plate with one displaced node is the kernel's values, C_ij(o) =
    alpha dV o_i o_j dx^2 / (r dx)^3 with alpha as the plan has it: a factor of
    r^2 rounded once and at most two roundings more (its products with o), 3
    units of 2^-53."""
    from decimal import Decimal, getcontext

    from paper_2105_06055_amd import binding
    getcontext().prec = 40
    dim, dx = len(body), 1.1e-3
    plan = binding.Plan(tuple(wl._grid_len(n, m) for n in body), body, dx, m * dx, E=72e9, dtype=torch.float64)
    at = tuple(n // 2 for n in body)
    u = torch.zeros((dim,) + body, dtype=torch.float64, device="cuda")
    u[(0,) + at] = 1.0
    L = plan.force(u).cpu().numpy()
    worst, h, alpha = 0.0, Decimal(dx), Decimal(plan.info["alpha"])
    for o in np.ndindex(*[2 * m + 1] * dim):
        o = tuple(q - m for q in o)[::-1]   # (x, y, z)
        r2 = sum(q * q for q in o)
        if not 0 < r2 <= m * m:
            continue
        node = tuple(a - q for a, q in zip(at, o[::-1]))   # the node whose bond o ends at the displaced one
        for d in range(dim):
            want = alpha * h ** dim * o[0] * o[d] * h * h / (Decimal(r2).sqrt() * h) ** 3
            got = Decimal(float(L[(d,) + node]))
            if want == 0:
                assert got == 0
            else:
                worst = max(worst, float(abs(got / want - 1)) * 2.0 ** 53)
    print(f"kernel values {body} m={m}: {worst:.2f} units of 2^-53", flush=True)
    assert worst <= 3.0, worst
    plan.close()
