"""Refined Helmholtz plans of 32-row chunks (more than 256 rows by default),
which eliminate once in float64: bitwise equal to the float64 plan, alone and
in the batch of a channel's u, v and w (513 rows, 512 faces), and the 16-row
chunks below the line, which refine, at the oracle's bar."""
import numpy as np
import pytest
import torch

import paper_2502_06296_amd as pf
import synth
from oracle import grid as ogrid
from oracle import poisson as op
from parity import TOL, check

pytestmark = pytest.mark.gpu
S = 1e-2


def _apply(ns, prec, rhs):
    plans = []
    for n in ns:
        plans.append(pf.pcr_prepare(*ogrid.zop(synth.tanh_faces(n, 2.0, 1.5), ogrid.DIRICHLET_CENTRE), S,
                                    precision=prec))
    u = [r.clone() for r in rhs]
    pf.pcr_apply_batched(plans, u)
    torch.cuda.synchronize()
    return u


@pytest.mark.parametrize("ns", [[257], [300], [512], [513, 513, 512], [1024, 257]])
def test_tall_refined_plans_are_the_float64_elimination(ns):
    print(f"helmholtz tall {ns}", flush=True)
    rhs = [torch.from_numpy(synth.normal01(60 + t, (n, 3, 64 * (1 + t)))).to("cuda:0") for t, n in enumerate(ns)]
    for a, b in zip(_apply(ns, "fp32_refine", rhs), _apply(ns, "fp64", rhs)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n", [129, 256])
def test_shorter_refined_plans_meet_the_oracle(n):
    r = torch.from_numpy(synth.normal01(70 + n, (n, 3, 128))).to("cuda:0")
    ref = op.solve_helmholtz(r.cpu().numpy(), synth.tanh_faces(n, 2.0, 1.5), S, ogrid.DIRICHLET_CENTRE)
    (u,) = _apply([n], "fp32_refine", [r])
    assert not np.array_equal(u.cpu().numpy(), _apply([n], "fp64", [r])[0].cpu().numpy())
    check(u.cpu().numpy(), ref, TOL["fp32_refine"], f"n={n}")
