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


# (float64, points, inverse, walls, behind x walls, slots, planes), the lines of
# a workgroup of the register engine, 0 for the LDS engine
Y_LINES = [
    ((True, 512, False, 0, False, 512, 512), 0), ((False, 128, False, 0, False, 512, 512), 0),
    # full workgroups, and narrow ones where those leave compute units idle
    ((False, 256, False, 0, False, 64, 64), 16), ((False, 1024, False, 0, False, 64, 256), 8),
    ((False, 1024, False, 0, False, 64, 16), 4), ((False, 3072, True, 0, False, 64, 11), 2),
    ((False, 3072, True, 0, False, 64, 22), 4), ((True, 3456, False, 1, False, 64, 10), 2),
    ((False, 384, False, 0, False, 1024, 512), 8), ((False, 512, True, 0, False, 512, 64), 8),
    ((False, 512, True, 0, False, 1024, 512), 16), ((False, 768, False, 0, False, 512, 40), 4),
    ((False, 768, False, 0, False, 1024, 256), 16), ((True, 768, False, 1, False, 256, 340), 4),
    ((True, 768, True, 0, False, 1024, 512), 8),
    # 48 slots
    ((False, 256, False, 1, False, 48, 1000), 8), ((False, 512, False, 1, False, 48, 512), 8),
    # cached float64 lines
    ((True, 1024, False, 0, False, 512, 32), 8), ((True, 2048, True, 0, False, 192, 40), 4),
    ((True, 2048, True, 0, False, 64, 16), 2), ((True, 1536, False, 0, False, 512, 30), 8),
    ((True, 1024, False, 0, False, 1024, 512), 8), ((True, 2048, True, 0, False, 1024, 128), 4),
    ((True, 1024, False, 1, False, 512, 32), 8), ((True, 2048, True, 1, False, 512, 16), 4),
    # faces, and the inverse behind x walls
    ((False, 2048, False, 3, False, 256, 128), 0), ((True, 2048, True, 3, False, 256, 128), 0),
    ((False, 1024, True, 3, False, 256, 128), 0), ((False, 1024, False, 3, False, 256, 128), 8),
    ((False, 1536, True, 3, False, 256, 128), 8), ((False, 512, True, 0, True, 256, 128), 0),
    ((False, 512, False, 0, True, 1024, 256), 16), ((False, 3072, True, 0, True, 64, 11), 0),
    ((False, 512, False, 3, False, 64, 128), 0), ((False, 512, False, 3, False, 512, 64), 8), ((False, 256, False, 1, False, 512, 16), 0),
    ((False, 256, True, 1, False, 512, 16), 16), ((False, 256, False, 1, False, 1024, 256), 16), ((True, 1024, True, 0, True, 256, 256), 0),
    ((False, 1536, True, 0, True, 256, 128), 8), ((True, 1536, True, 0, True, 256, 128), 8),
]


@pytest.mark.parametrize("case,lines", Y_LINES)
def test_y_transform_lines_are_the_faster_ones(case, lines):
    rule = _rule("_ZN2pf7y_linesEbibibii", C.c_bool, C.c_int, C.c_bool, C.c_int, C.c_bool, C.c_int, C.c_int)
    assert rule(*case) == lines


# (pass, float64, points, line pairs), the line pairs of a workgroup of the
# register engine, 0 for the LDS engine
FWD, INV, RESID, DIV = 0, 1, 2, 3
X_LINES = [
    ((FWD, False, 256, 1 << 16), 0), ((FWD, False, 512, 1 << 18), 0), ((FWD, False, 768, 1 << 16), 4),
    ((FWD, True, 1024, 1 << 17), 0), ((FWD, True, 2048, 1 << 15), 0), ((FWD, True, 3072, 1 << 15), 0),
    ((FWD, True, 1536, 1 << 15), 2), ((FWD, True, 3456, 1 << 15), 1),
    ((FWD, False, 1024, 513), 4), ((FWD, False, 1024, 512), 2), ((FWD, False, 3200, 100), 1),
    ((INV, False, 512, 1 << 18), 0), ((INV, False, 384, 1 << 16), 8), ((INV, False, 2048, 200), 1),
    ((INV, True, 2048, 1 << 15), 0), ((INV, True, 3456, 1 << 15), 1),
    ((DIV, True, 192, 1 << 14), 0), ((DIV, True, 512, 1 << 12), 4), ((DIV, True, 512, 1 << 14), 8),
    ((DIV, False, 1024, 1 << 11), 2), ((DIV, True, 1024, 1 << 14), 4), ((DIV, True, 768, 1 << 11), 4),
    ((RESID, False, 384, 1 << 14), 8), ((RESID, False, 512, 1 << 17), 4), ((RESID, False, 768, 1 << 14), 4),
    ((RESID, False, 1024, 1 << 17), 4), ((RESID, False, 1536, 1 << 16), 0), ((RESID, False, 2048, 1 << 15), 2),
]


@pytest.mark.parametrize("case,lines", X_LINES)
def test_x_transform_lines_are_the_faster_ones(case, lines):
    rule = _rule("_ZN2pf7x_linesEibil", C.c_int, C.c_bool, C.c_int, C.c_long)
    assert rule(*case) == lines


@pytest.mark.parametrize("resident,tiles", [
    (512, [13 * 192, 9 * 128, 5 * 64]), (256, [17 * 256, 13 * 96, 9 * 64, 5 * 64, 17 * 192]), (1024, [300, 200, 500]),
    (256, [100000] + [64] * 15), (512, [1] * 16), (256, [4000] * 16)])
def test_grouped_persistent_shares_fit_one_round(resident, tiles):
    fn = N.lib()._ZN2pf14z_group_sharesEliPKlPj
    fn.restype = None
    n = len(tiles)
    share = (C.c_uint * n)()
    fn(C.c_long(resident), C.c_int(n), (C.c_long * n)(*tiles), share)
    assert sum(share) <= resident
    assert all(1 <= s <= t for s, t in zip(share, tiles))
    # nothing is left over, and no workgroup has more than one tile above the
    # even split of what the jobs of one workgroup leave
    assert sum(share) == min(resident, sum(tiles))
    even = -(-sum(tiles) // (resident - n))
    assert max(-(-t // s) for s, t in zip(share, tiles)) <= even + 1
