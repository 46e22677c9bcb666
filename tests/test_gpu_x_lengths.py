"""Every x length in every precision against the CPU oracle at the bars of the
other parity tests: the x transforms and the residual on both engines, single
and grouped, with periodic and walled y (the residual's ghost rows), and the
tuner's x shapes of the lengths that have them."""
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
LENGTHS = [64, 96, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048, 3072, 3200, 3456]


@pytest.mark.parametrize("nx", LENGTHS)
@pytest.mark.parametrize("ybc", [0, 1, 2])
@pytest.mark.parametrize("prec", ["fp64", "fp32_refine", "fp32"])
def test_x_length_matches_oracle(nx, ybc, prec):
    ny, nz = 64, 9
    f, zf = synth.channel_rhs(700 + nx, nx, ny, nz, beta=1.5)
    ref = op.solve_poisson(f, zf, LX, LY, ybc=ybc)
    plan = pf.poisson_plan(nx, ny, nz, LX, LY, 2.0, 1.5, zf=zf, precision=prec, ybc=ybc, tuned=False)
    rhs = torch.from_numpy(f).to("cuda:0")
    p = torch.empty_like(rhs)
    for v in range(autotune.transform_shape_count(plan)):
        if autotune.set_variant(plan, autotune.STAGE_XFWD, v):
            pf.poisson_solve(plan, rhs, p)
            torch.cuda.synchronize()
            check(p.cpu().numpy(), ref, TOL[prec], f"{prec} nx={nx} ybc={ybc} shape {v}")


def test_grouped_x_lengths_match_oracle():
    plans, rhs, out, ref = [], [], [], []
    for t, nx in enumerate(LENGTHS):
        ny, nz = (64, 96)[t % 2], 6 + t % 3
        f, zf = synth.channel_rhs(800 + t, nx, ny, nz, beta=1.2)
        ref.append(op.solve_poisson(f, zf, LX, LY))
        plans.append(pf.poisson_plan(nx, ny, nz, LX, LY, 2.0, 1.2, zf=zf, precision="fp32_refine", tuned=False))
        rhs.append(torch.from_numpy(f).to("cuda:0"))
        out.append(torch.empty_like(rhs[-1]))
    pf.poisson_solve_batched(plans, rhs, out)
    torch.cuda.synchronize()
    for p, r, nx in zip(out, ref, LENGTHS):
        check(p.cpu().numpy(), r, TOL["fp32_refine"], f"grouped nx={nx}")
