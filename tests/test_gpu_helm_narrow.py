"""Refined Helmholtz plans whose chunks are narrower than a wave, which
eliminate once in float64: at the row counts on both sides of the default's
line (512) and on explicit shapes, against the float64 plan of the same shape
(the same elimination on the same tables: bitwise), and in batches that mix
both kinds of chunk (each field as in a call of its own: bitwise)."""
import numpy as np
import pytest
import torch

import paper_2502_06296_amd as pf
import synth
from oracle import grid as ogrid
from oracle import poisson as op
from paper_2502_06296_amd import autotune
from parity import TOL, check

pytestmark = pytest.mark.gpu
S = 1e-2


def _plan(n, prec):
    al, ga, ex = ogrid.zop(synth.tanh_faces(n, 2.0, 1.5), ogrid.DIRICHLET_CENTRE)
    return pf.pcr_prepare(al, ga, ex, S, precision=prec)


def _rhs(n, ny, nx, seed):
    return torch.from_numpy(synth.normal01(seed, (n, ny, nx))).to("cuda:0")


@pytest.mark.parametrize("n,shape", [(512, None), (513, None), (777, None), (1023, None), (1024, None),
                                     (40, (8, 32)), (250, (16, 16)), (512, (32, 32))])
def test_narrow_refined_plan_is_the_float64_elimination(n, shape):
    print(f"helmholtz n={n} shape={shape}", flush=True)
    r = _rhs(n, 3, 192, 31)
    got = {}
    for prec in ("fp64", "fp32_refine"):
        plan = _plan(n, prec)
        if shape:
            assert autotune.set_pcr_shape([plan], *shape)
        u = r.clone()
        pf.pcr_apply(plan, u)
        torch.cuda.synchronize()
        got[prec] = u.cpu().numpy()
    ref = op.solve_helmholtz(r.cpu().numpy(), synth.tanh_faces(n, 2.0, 1.5), S, ogrid.DIRICHLET_CENTRE)
    check(got["fp32_refine"], ref, TOL["fp32_refine"], f"n={n}")
    if n > 512 or shape:
        assert np.array_equal(got["fp32_refine"], got["fp64"])


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32_refine"])
def test_batch_of_wide_and_narrow_chunks(prec):
    ns = [300, 600, 512, 1024, 513]
    plans = [_plan(n, prec) for n in ns]
    dt = torch.float32 if prec == "fp32" else torch.float64
    rhs = [_rhs(n, 2 + t, 64 * (1 + t % 2), 40 + t).to(dt) for t, n in enumerate(ns)]
    alone = [r.clone() for r in rhs]
    for p, u in zip(plans, alone):
        pf.pcr_apply(p, u)
    both = [r.clone() for r in rhs]
    pf.pcr_apply_batched(plans, both)
    torch.cuda.synchronize()
    for n, a, b in zip(ns, alone, both):
        assert torch.equal(a, b), n
