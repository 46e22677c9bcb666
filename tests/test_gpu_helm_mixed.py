"""Refined Helmholtz batches of 32-row chunks on both sides of 512 rows (a
channel's u, v and w of 513 rows among them), which share one launch: each
field as in a call of its own (bitwise) and at the oracle's bar."""
import pytest
import torch

import paper_2502_06296_amd as pf
import synth
from oracle import grid as ogrid
from oracle import poisson as op
from parity import TOL, check

pytestmark = pytest.mark.gpu
S = 1e-2


@pytest.mark.parametrize("rows,nx,ny", [([513, 513, 512], 64, 3), ([512, 513], 320, 9), ([1024, 257, 700, 300], 128, 4),
                                        ([257] + [600] * 15, 64, 2)])
def test_both_kinds_of_chunk_in_one_launch(rows, nx, ny):
    print(f"helmholtz mixed {rows} {nx}x{ny}", flush=True)
    plans, rhs = [], []
    for t, n in enumerate(rows):
        plans.append(pf.pcr_prepare(*ogrid.zop(synth.tanh_faces(n, 2.0, 1.5), ogrid.DIRICHLET_CENTRE), S,
                                    precision="fp32_refine"))
        rhs.append(torch.from_numpy(synth.normal01(80 + t, (n, ny + t % 2, nx))).to("cuda:0"))
    alone, both = [r.clone() for r in rhs], [r.clone() for r in rhs]
    for p, u in zip(plans, alone):
        pf.pcr_apply(p, u)
    pf.pcr_apply_batched(plans, both)
    torch.cuda.synchronize()
    for n, r, a, b in zip(rows, rhs, alone, both):
        assert torch.equal(a, b), n
        ref = op.solve_helmholtz(r.cpu().numpy(), synth.tanh_faces(n, 2.0, 1.5), S, ogrid.DIRICHLET_CENTRE)
        check(b.cpu().numpy(), ref, TOL["fp32_refine"], f"n={n}")
