"""The projection correction with its planes cut into chunks (small planes):
plane counts around the chunk height, against the CPU oracle at the bars of
test_gpu_projection.py."""
import numpy as np
import pytest

from oracle import projection as oproj
from test_gpu_projection import LX, LY, TOL, _inputs, _project_gpu
import synth
from parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [4, 7, 8, 9, 16, 17, 65])
@pytest.mark.parametrize("c", [0.0, 1e-3])
def test_chunked_correction_matches_oracle(nz, c):
    nx, ny = 96, 64
    zf = synth.tanh_faces(nz, 2.0, 1.5)
    u, v, w, p = _inputs(80 + nz, nx, ny, nz)
    ref = oproj.project(u, v, w, p, zf, LX, LY, 0.37, c)
    got = _project_gpu(u, v, w, p, zf, 1.5, "fp64", 0.37, c)
    for name, g, r in zip(("u", "v", "w", "p", "phi"), got, ref):
        check(g, r, TOL["fp64"], f"nz={nz} {name}")
