"""Rules that choose a launch from sizes, on the CPU: each against the side that was
measured to be the faster one."""
import pytest

from tests import host_plan

FP32, FP64 = 4, 8


# grid, bytes, iterations, rows of both systems, work items of e_z and h_z, planes per
# chunk, whether several iterations per pass were the faster way
IMPLICIT = [
    ("30x26x100 taper", FP32, 15, 2920 + 4004, 22, 26, 1, False),
    ("30x26x100 taper", FP64, 31, 2920 + 4004, 22, 26, 1, False),
    ("60x60x400 taper", FP64, 31, 153688 + 169328, 295, 336, 1, False),
    ("60x60x400 taper", FP32, 15, 153688 + 169328, 283, 309, 1, False),
    ("60x60x400", FP64, 31, 1392400 + 1436400, 210, 210, 6, True),
    ("60x60x400", FP32, 15, 1392400 + 1436400, 210, 210, 4, True),
    ("24x24x48", FP32, 15, 25392 + 27072, 23, 24, 1, False),
    ("24x24x48", FP64, 31, 25392 + 27072, 23, 24, 1, False),
    ("40x40x200 jaws", FP32, 15, 241488 + 253120, 160, 160, 2, False),
    ("80x80x64", FP64, 31, 399424 + 403200, 216, 216, 3, False),
    ("33x27x941 jaws", FP64, 31, 622144 + 671220, 182, 182, 5, False),
    ("64x64x256 wide", FP32, 6, 1016064 + 1044480, 220, 220, 3, False),
    ("64x64x256 fine", FP32, 46, 1016064 + 1044480, 220, 220, 3, True),
    ("30x26x100 fine", FP32, 55, 72500 + 77220, 58, 60, 1, False),
    ("200x8x200", FP32, 15, 278600 + 318400, 200, 200, 4, False),
    ("8x200x200", FP32, 15, 278600 + 318400, 168, 192, 1, True),
    ("104x89x758 taper", FP32, 15, 821184 + 871884, 210, 218, 5, True),
    ("160x160x512 jaws", FP32, 15, 10333728 + 10439680, 195, 180, 33, True),
    ("160x160x512 jaws", FP64, 31, 10333728 + 10439680, 220, 216, 41, True),
    ("200x180x700 taper", FP32, 15, 1366520 + 1424248, 155, 165, 10, True),
]


@pytest.mark.parametrize("case", IMPLICIT, ids=lambda c: "%s-%d-%d" % c[:3])
def test_implicit_solves_take_the_faster_way(case):
    _, rb, iters, rows, ie, ih, xc, passes = case
    # the library knows the rows of e_z and takes as many for h_z
    for r in (rows, int(0.94 * rows)):
        assert bool(host_plan.lib().implicit(rb, iters, 5 if rb == FP32 else 4, r, ie, ih, xc)) == passes
