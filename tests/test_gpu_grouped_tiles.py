"""Grouped persistent z solves of several jobs that share a launch, whose
shares of the resident workgroups are fewer than their tiles, so that every
workgroup walks several: bitwise equal to the solves one by one."""
import pytest
import torch

import paper_2502_06296_amd as pf
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz,planes", [
    (384, [(256, 256), (192, 256), (64, 128)]), (100, [(256, 256), (192, 192), (256, 128), (64, 64)]),
    (1024, [(128, 96), (64, 64), (96, 64)])])
def test_several_jobs_of_several_tiles_equal_the_single_solves(nz, planes):
    plans, rhs, one, out = [], [], [], []
    for t, (nx, ny) in enumerate(planes):
        print(f"grouped tiles {nx}x{ny}x{nz}", flush=True)
        plans.append(pf.poisson_plan(nx, ny, nz, 6.0, 3.0, 2.0, 1.4, precision="fp32_refine", tuned=False))
        rhs.append(torch.from_numpy(synth.uniform_pm1(nz + t, (nz, ny, nx))).to("cuda:0"))
        one.append(torch.empty_like(rhs[-1]))
        out.append(torch.full_like(rhs[-1], 5.0))
        pf.poisson_solve(plans[-1], rhs[-1], one[-1])
    pf.poisson_solve_batched(plans, rhs, out)
    torch.cuda.synchronize()
    for a, b, plane in zip(one, out, planes):
        assert torch.equal(a, b), plane
