"""The transform chains in their default forms, on plans that would run the
direct sums: the tests below once more with those switched off.  Plans with
unequal spacings, longer horizons or weights in 3D run this code: the x passes
(mixed-radix lengths too) and the (y, z) correlation, the FP64 chained Verlet
epilogue, the weighted plate's chain with the failure rule, the energies, the
adjoints and the damage count."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2105_06055_amd import workloads as wl

from test_gpu_autograd import (test_checkpoint_recompute_is_bitwise_fp32, test_checkpointed_rollout_fd_and_oracle,  # noqa: F401
                               test_pdforce_function_gradcheck_directions, test_rollout_load_gradient)
from test_gpu_dynamics import (test_clamped_layer_and_body_force, test_fracture_subcase_damage_bit_exact,  # noqa: F401
                               test_lps_block_dynamics, test_lps_clamped_layer_body_force_multistep,
                               test_nonfinite_state_reports_numeric, test_plate_trajectory_100_steps,
                               test_regrouped_steps_against_single_steps, test_shadow_energy_conserved_fp64)
from test_gpu_force import (test_bb2d_integrity_weights_and_energy, test_bb2d_masked_ragged, test_bb2d_scale_weights,  # noqa: F401
                            test_bb3d_masked, test_damage_index_bit_exact, test_energy_density_large_displacement,
                            test_influence_one, test_lps3d_long_horizons_all_paths, test_lps3d_ragged_voids,
                            test_mixed_radix_x_bb2d, test_mixed_radix_x_lps3d_all_paths,
                            test_mixed_radix_x_weighted_energy_2d, test_yz_direct_tiles)
from test_gpu_nbb import (test_nbb2d_masked_ragged, test_nbb2d_rigid_rotation_zero_force, test_nbb3d_masked,  # noqa: F401
                          test_nbb3d_rigid_rotation_zero_force, test_nbb3d_yz_pass_against_y_transform_path)
from test_gpu_routes import _passes, test_unweighted_plate_adjoint_and_energies  # noqa: F401
from test_gpu_static_adjoint import (test_force_adjoint_scale_weights, test_static_bb2d_clamped,  # noqa: F401
                                     test_static_lps_cube_void, test_verlet_adjoint_step_chain)
from test_gpu_verlet_errors import test_state_after_nonfinite_energy  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def transforms(monkeypatch):
    """Every plan's default kernel choice without the direct sums."""
    from paper_2105_06055_amd import binding
    monkeypatch.setattr(binding.Plan, "LASTAXIS", dict(binding.Plan.LASTAXIS, auto=binding.Plan.LASTAXIS["transform"]))
    init = binding.Plan.__init__

    def with_transforms(self, *args, **kw):
        init(self, *args, **kw)
        self.set_lastaxis("auto")

    monkeypatch.setattr(binding.Plan, "__init__", with_transforms)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_passes_of_this_module(dtype):
    """What the fixture makes the calls run: no direct sums, in 3D the (y, z)
    correlation, in FP64 the chained inner steps."""
    from paper_2105_06055_amd import binding

    def plan_of(body, **kw):
        return binding.Plan(tuple(wl._grid_len(n, 3) for n in body), body, 1e-3, 3e-3, E=72e9, nu=0.3, rho=2440.0,
                            dtype=dtype, **kw)

    def state(plan, **kw):
        z = torch.zeros((plan.dim,) + plan.body, dtype=dtype, device="cuda")
        return dict({"u": z, "v": z + 1.0, "F": z.clone(), "step": 0}, **kw)

    block = plan_of((20, 21, 22), model="lps")
    names = _passes(block, lambda: block.verlet(state(block), 1e-8, 4))
    assert not any(n.startswith("dir") for n in names) and any(n.startswith("yzconv") for n in names), names
    assert ("xinvfwd_3_3" in names) == (dtype == torch.float64), names
    block.close()
    plate = plan_of((40, 50), weight="integrity", G0=3.8)
    lam, W = torch.ones(plate.body, dtype=torch.uint8, device="cuda"), torch.zeros(plate.body, dtype=dtype, device="cuda")
    names = _passes(plate, lambda: (plate.verlet(state(plate, lam=lam, W=W), 1e-8, 2), plate.damage_index(lam)))
    assert not any(n.startswith(("dir", "damage2")) for n in names) and "energy_direct" in names, names
    plate.close()
