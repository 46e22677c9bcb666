"""Every y length in every precision and with every y boundary, and with x
walls, against the CPU oracle at the bars of the other parity tests: the
lengths the register engine takes, those the LDS engine keeps, and the
48-slot planes that take half the columns per workgroup."""
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
LENGTHS = [64, 96, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048, 3072, 3200, 3456]
YBC = {"periodic": ogrid.Y_PERIODIC, "walls": ogrid.Y_WALLS, "dirichlet": ogrid.Y_DIRICHLET, "faces": ogrid.Y_FACES}


@pytest.mark.parametrize("ny", LENGTHS)
@pytest.mark.parametrize("ybc,xbc", [("periodic", 0), ("walls", 0), ("dirichlet", 0), ("periodic", 1)])
@pytest.mark.parametrize("prec", ["fp64", "fp32_refine", "fp32"])
def test_y_length_matches_oracle(ny, ybc, xbc, prec):
    nx, nz = 64, 5
    f, zf = synth.channel_rhs(500 + ny, nx, ny, nz, beta=1.5)
    ref = op.solve_poisson(f, zf, LX, LY, ybc=YBC[ybc], xbc=xbc)
    plan = pf.poisson_plan(nx, ny, nz, LX, LY, 2.0, 1.5, zf=zf, precision=prec, ybc=ybc,
                           xbc="walls" if xbc else "periodic", tuned=False)
    rhs = torch.from_numpy(f).to("cuda:0")
    p = torch.empty_like(rhs)
    pf.poisson_solve(plan, rhs, p)
    torch.cuda.synchronize()
    check(p.cpu().numpy(), ref, TOL[prec], f"{prec} ny={ny} {ybc} xbc={xbc}")


def _faces(nx, ny, ybc, xbc, prec):
    nz, s = 5, 1e-2
    zf = synth.tanh_faces(nz, 2.0, 1.5)
    r = synth.normal01(900 + ny, (nz, ny, nx))
    xc = ogrid.X_FACES if xbc == "faces" else 0
    ref = op.solve_helmholtz3d(r, zf, s, ogrid.DIRICHLET_CENTRE, LX, LY, ybc=YBC[ybc], xbc=xc)
    plan = pf.helmholtz3d_plan(nx, ny, nz, "dirichlet_centre", s, LX, LY, 2.0, 1.5, zf=zf, precision=prec,
                               ybc=ybc, xbc=xbc)
    rt = torch.from_numpy(r).to("cuda:0")
    u = torch.empty_like(rt)
    pf.helmholtz3d_solve(plan, rt, u)
    torch.cuda.synchronize()
    check(u.cpu().numpy(), ref, TOL[prec], f"{prec} {nx}x{ny} {ybc} {xbc}")


@pytest.mark.parametrize("ny2", LENGTHS)
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_y_faces_length_matches_oracle(ny2, prec):
    _faces(64, ny2 // 2, "faces", "periodic", prec)


@pytest.mark.parametrize("ny", [512, 768, 1024, 2048])
@pytest.mark.parametrize("ybc", ["periodic", "walls"])
@pytest.mark.parametrize("prec", ["fp64", "fp32_refine", "fp32"])
def test_48_slots_match_oracle(ny, ybc, prec):
    _faces(48, ny, ybc, "faces", prec)
