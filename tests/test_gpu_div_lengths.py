"""The projection's divergence pass at every x length (both transform engines),
with periodic y and with y walls, on the fewest planes and on an odd number,
against the CPU oracle at the bars of the projection's parity test."""
import numpy as np
import pytest
import torch

import paper_2502_06296_amd as pf
import synth
from oracle import projection as oproj
from parity import check

pytestmark = pytest.mark.gpu
LX, LY = 2 * np.pi, np.pi
TOL = {"fp64": 1e-12, "fp32_refine": 1e-10, "fp32": 1e-5}


@pytest.mark.parametrize("nx", [64, 96, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048, 3072, 3200, 3456])
@pytest.mark.parametrize("ybc,nz", [(0, 4), (0, 9), (1, 9)])
@pytest.mark.parametrize("prec", ["fp64", "fp32_refine", "fp32"])
def test_divergence_length_matches_oracle(nx, ybc, nz, prec):
    print(f"divergence {prec} nx={nx} nz={nz} ybc={ybc}", flush=True)
    ny, beta, gdt, c = 64, 1.5, 0.37, 1e-3
    zf = synth.tanh_faces(nz, 2.0, beta)
    u, v, w, p = (synth.uniform_pm1(900 + nx + s, (nz - (s == 2), ny, nx)) for s in range(4))
    ref = oproj.project(u, v, w, p, zf, LX, LY, gdt, c, ybc=ybc)
    plan = pf.poisson_plan(nx, ny, nz, LX, LY, 2.0, beta, zf=zf, precision=prec, ybc=ybc, tuned=False)
    t = [torch.from_numpy(a).to("cuda:0") for a in (u, v, w, p)]
    phi = torch.empty_like(t[0])
    pf.poisson_project(plan, *t, phi, gdt, c)
    torch.cuda.synchronize()
    for name, g, r in zip(("u", "v", "w", "p", "phi"), (*t, phi), ref):
        check(g.cpu().numpy(), r, TOL[prec], name)
