"""The singular (0,0) mode inside the y forward (plane means) and the z solve
(its pinned solve): a right-hand side dominated by its plane means, at row
counts around the 64 lanes of the solve and its 16 rows a lane, with the
smallest workgroups that z-solve variants launch, against the CPU oracle at
the bars of the other parity tests."""
import numpy as np
import pytest
import torch

import paper_2502_06296_amd as pf
import synth
from oracle import poisson as op
from paper_2502_06296_amd import autotune
from parity import TOL, check

pytestmark = pytest.mark.gpu
LX, LY = 2 * np.pi, np.pi


def _profile_rhs(seed, nx, ny, nz, beta):
    zf = synth.tanh_faces(nz, 2.0, beta)
    f = 0.05 * synth.uniform_pm1(seed, (nz, ny, nx)) + synth.uniform_pm1(seed + 1, (nz, 1, 1))
    return f, zf


@pytest.mark.parametrize("nz", [4, 5, 17, 63, 64, 65, 130, 1023, 1024])
@pytest.mark.parametrize("prec", ["fp64", "fp32_refine", "fp32"])
def test_plane_mean_profile_matches_oracle(nz, prec):
    nx, ny = 64, 96
    f, zf = _profile_rhs(300 + nz, nx, ny, nz, 1.5)
    ref = op.solve_poisson(f, zf, LX, LY)
    plan = pf.poisson_plan(nx, ny, nz, LX, LY, 2.0, 1.5, zf=zf, precision=prec, tuned=False)
    rhs = torch.from_numpy(f).to("cuda:0")
    p = torch.full_like(rhs, 3.0)
    for v in [None] + autotune.zsolve_variants(plan):
        if v is not None and not autotune.set_zsolve_variant(plan, v):
            continue
        pf.poisson_solve(plan, rhs, p)
        torch.cuda.synchronize()
        got = p.cpu().numpy()
        check(got, ref, TOL[prec], f"{prec} nz={nz} variant {v}")
        check(got.mean(axis=(1, 2)), ref.mean(axis=(1, 2)), TOL[prec], "plane means")


@pytest.mark.parametrize("prec", ["fp64", "fp32_refine"])
@pytest.mark.parametrize("ybc,xbc", [("walls", "periodic"), ("periodic", "walls"), ("walls", "walls")])
def test_plane_mean_profile_with_walls(ybc, xbc, prec):
    nx, ny, nz = 64, 192, 70
    f, zf = _profile_rhs(31, nx, ny, nz, 1.2)
    code = {"periodic": 0, "walls": 1}
    ref = op.solve_poisson(f, zf, LX, LY, ybc=code[ybc], xbc=code[xbc])
    plan = pf.poisson_plan(nx, ny, nz, LX, LY, 2.0, 1.2, zf=zf, precision=prec, ybc=ybc, xbc=xbc)
    rhs = torch.from_numpy(f).to("cuda:0")
    p = torch.empty_like(rhs)
    pf.poisson_solve(plan, rhs, p)
    torch.cuda.synchronize()
    check(p.cpu().numpy(), ref, TOL[prec], f"{prec} {ybc} {xbc}")
