"""The y transforms on both sides of the workgroup counts at which their lines
per workgroup, or the engine, change: against the CPU oracle at the last
narrow and the first full launch, and, where that takes a large field, float32
storage against float64 (both meet the oracle's bars, so two solutions differ
by the sum of the bars at most)."""
import numpy as np
import pytest
import torch

import paper_2502_06296_amd as pf
import synth
from oracle import grid as ogrid
from oracle import poisson as op
from parity import TOL, check

pytestmark = pytest.mark.gpu
LX, LY = 2 * np.pi, np.pi
YBC = {"periodic": ogrid.Y_PERIODIC, "walls": ogrid.Y_WALLS, "dirichlet": ogrid.Y_DIRICHLET}


def _solve(nx, ny, nz, prec, f, zf, **kw):
    plan = pf.poisson_plan(nx, ny, nz, LX, LY, 2.0, 1.5, zf=zf, precision=prec, tuned=False, **kw)
    p = torch.full_like(f, 3.0)
    pf.poisson_solve(plan, f, p)
    torch.cuda.synchronize()
    return p


# 64 slots: 4 nz workgroups of 8 lines, 8 nz of 4 lines
@pytest.mark.parametrize("prec,ny,edge", [
    ("fp32", 1024, 32), ("fp32", 1536, 32), ("fp32", 2048, 16), ("fp32", 3200, 16), ("fp64", 1024, 32),
    ("fp64", 768, 48), ("fp64", 3456, 16), ("fp64", 2048, 16)])
@pytest.mark.parametrize("ybc,xbc", [("periodic", 0), ("walls", 0), ("dirichlet", 0), ("periodic", 1)])
@pytest.mark.parametrize("past", [0, 1])
def test_last_narrow_and_first_full_launch_match_oracle(prec, ny, edge, ybc, xbc, past):
    nx, nz = 64, edge + past
    print(f"y workgroups {prec} {nx}x{ny}x{nz} {ybc} xbc={xbc}", flush=True)
    f, zf = synth.channel_rhs(40 + ny, nx, ny, nz, beta=1.5)
    ref = op.solve_poisson(f, zf, LX, LY, ybc=YBC[ybc], xbc=xbc)
    p = _solve(nx, ny, nz, prec, torch.from_numpy(f).to("cuda:0"), zf, ybc=ybc, xbc="walls" if xbc else "periodic")
    check(p.cpu().numpy(), ref, TOL[prec], f"{prec} ny={ny} nz={nz} {ybc} xbc={xbc}")


@pytest.mark.parametrize("nx,ny,nz", [(1024, 512, 62), (1024, 512, 66), (1024, 768, 126), (1024, 768, 130)])
@pytest.mark.parametrize("ybc", ["periodic", "walls"])
def test_wide_launches_agree_between_precisions(nx, ny, nz, ybc):
    print(f"y workgroups {nx}x{ny}x{nz} {ybc}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(nz)
    f = torch.rand((nz, ny, nx), dtype=torch.float64, device="cuda:0", generator=g) - 0.5
    p64, p32 = (_solve(nx, ny, nz, prec, f, None, ybc=ybc) for prec in ("fp64", "fp32"))
    d = (p32 - p64).abs_()
    tol = TOL["fp64"] + TOL["fp32"]
    assert float(d.max() / p64.abs().max()) < tol
    assert float(d.norm() / p64.norm()) < tol
