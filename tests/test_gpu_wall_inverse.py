"""The wall inverses along y, with every row read once or twice by length, under
x walls too (every slot its own mode), against the CPU oracle at the bars of
the other parity tests."""
import numpy as np
import pytest
import torch

import paper_2502_06296_amd as pf
import synth
from oracle import poisson as op
from parity import TOL, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny", [256, 384, 512, 768, 1024, 2048, 3456])
@pytest.mark.parametrize("ybc,xbc", [(1, 1), (2, 1), (1, 2), (2, 2)])
@pytest.mark.parametrize("prec", ["fp64", "fp32_refine", "fp32"])
def test_wall_inverse_with_x_walls_matches_oracle(ny, ybc, xbc, prec):
    print(f"wall inverse {prec} ny={ny} ybc={ybc} xbc={xbc}", flush=True)
    nx, nz, lx, ly = 64, 5, 2 * np.pi, np.pi
    f, zf = synth.channel_rhs(600 + ny, nx, ny, nz, beta=1.5)
    ref = op.solve_poisson(f, zf, lx, ly, ybc=ybc, xbc=xbc)
    plan = pf.poisson_plan(nx, ny, nz, lx, ly, 2.0, 1.5, zf=zf, precision=prec, ybc=ybc, xbc=xbc, tuned=False)
    rhs = torch.from_numpy(f).to("cuda:0")
    p = torch.empty_like(rhs)
    pf.poisson_solve(plan, rhs, p)
    torch.cuda.synchronize()
    check(p.cpu().numpy(), ref, TOL[prec], f"{prec} ny={ny} ybc={ybc} xbc={xbc}")
