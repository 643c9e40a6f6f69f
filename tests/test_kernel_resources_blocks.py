"""Occupancy floors of the kernels on the main path (waves per SIMD, gfx950, from the
compiler's resource report): the shared forward walks and their normalisers, the block
gather and its lists, the registration in step, the FP64 motion derivative, the robust
weights, superpixels and the convolutions' gradients."""
import os

import pytest

from test_kernel_resources import HIPCC, occupancies

FLOORS = {
    "pvr_forward.hip": {"_Z17k_simulate_planesIfE": 7, "_Z17k_simulate_planesIdE": 3},
    "pvr_plan.hip": {"_Z20k_normalisers_planesIfE": 7, "_Z20k_normalisers_planesIdE": 4,
                     "_Z11k_adj_listsILi6E": 6, "_Z11k_adj_listsILi8E": 4},
    "pvr_adjoint.hip": {"_Z15k_gather_blocksIfLb1ELb0E": 6, "_Z15k_gather_blocksIfLb0ELb0E": 7,
                        "_Z15k_gather_blocksIfLb1ELb1E": 5, "_Z15k_gather_blocksIfLb0ELb1E": 7,
                        "_Z15k_gather_blocksIdLb1ELb0E": 3, "_Z15k_gather_blocksIdLb0ELb0E": 4},
    "pvr_register.hip": {"_Z10k_reg_evalILi0E": 8, "_Z10k_reg_evalILi1E": 7, "_Z10k_reg_grad": 4},
    "pvr_grad.hip": {"_Z19k_grad_theta_planes": 2},
    "pvr_em.hip": {"_Z10k_em_estep": 8, "_Z12k_em_patchesILi256ELi256E": 7},
    "pvr_slic.hip": {"_Z13k_slic_gather": 8, "_Z13k_slic_updateILb1E": 8},
    "pvr_cnn.hip": {"_Z12k_wgrad_tile": 4},
}


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("src", sorted(FLOORS))
def test_main_path_kernels_keep_their_occupancy(src):
    occ = occupancies(src)
    for prefix, floor in FLOORS[src].items():
        got = [v for k, v in occ.items() if k.startswith(prefix)]
        assert got, f"kernel {prefix} not found in {src}"
        assert min(got) >= floor, f"{prefix}: occupancy {min(got)} < {floor} waves/SIMD"
