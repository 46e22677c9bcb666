"""The rules that choose a launch by size, read from the library on the host:
each row is a grid on which both sides of a rule were timed, with the side
that was faster."""
import ctypes as C

import pytest

from paper_2502_06296_amd import _native as N


def _rule(name, *types):
    fn = getattr(N.lib(), name)
    fn.restype, fn.argtypes = C.c_int, list(types)
    return fn


# (nx, ny, nz), float64, x walls, the z-solve shape
Z_DEFAULTS = [
    ((64, 64, 64), True, False, 41), ((256, 256, 128), True, False, 41),
    ((256, 256, 384), True, False, 18), ((384, 256, 300), True, False, 18), ((512, 256, 192), True, False, 18),
    # 2^25 points: the field leaves the last-level cache
    ((512, 256, 256), True, False, 40), ((384, 256, 384), True, False, 40), ((512, 256, 512), True, False, 40),
    ((256, 128, 1024), True, False, 38), ((256, 256, 768), True, False, 38), ((384, 192, 1024), True, False, 38),
    ((512, 512, 128), True, False, 40),
    # x walls: two passes of every tile
    ((64, 64, 64), True, True, 41), ((128, 128, 16), True, True, 24), ((128, 128, 64), True, True, 26),
    ((256, 256, 16), True, True, 24), ((256, 256, 128), True, True, 18), ((256, 256, 768), True, True, 38),
    ((256, 256, 256), False, False, 41), ((512, 512, 16), False, False, 42), ((512, 512, 256), False, False, 41),
    ((128, 128, 16), False, True, 42), ((512, 512, 16), False, True, 24), ((512, 512, 30), False, True, 42),
    ((512, 512, 160), False, True, 41), ((512, 256, 192), False, True, 39), ((512, 512, 256), False, True, 39),
    ((1024, 512, 192), False, True, 41), ((512, 512, 384), False, True, 41),
]


@pytest.mark.parametrize("grid,fp64,xwalls,shape", Z_DEFAULTS)
def test_default_z_solve_is_the_faster_one(grid, fp64, xwalls, shape):
    rule = _rule("_ZN2pf22zsolve_default_variantEiiibb", C.c_int, C.c_int, C.c_int, C.c_bool, C.c_bool)
    assert rule(*grid, fp64, xwalls) == shape
