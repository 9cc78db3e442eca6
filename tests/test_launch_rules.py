"""Rules that choose a launch from sizes, on the CPU: each against the side that was
measured to be the faster one."""
import random
import time

import numpy as np
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


# nr, nz, bytes, rows per chunk measured within a few percent of the best
RZ = [
    (1000, 18183, FP32, (84, 112, 126)), (1000, 18183, FP64, (84, 167)), (500, 9000, FP32, (27, 28)),
    (500, 9000, FP64, (42,)), (700, 14000, FP32, (59, 64)), (700, 14000, FP64, (88, 92)), (1000, 4000, FP32, (24, 36)),
    (1000, 4000, FP64, (36,)), (200, 18183, FP64, (34,)), (333, 4001, FP32, (12,)), (333, 4001, FP64, (12,)),
    (300, 300, FP32, (12,)), (300, 300, FP64, (12,)), (60, 700, FP32, (12, 13)), (5000, 100, FP64, (12,)),
    (100000, 40, FP32, (33,)), (100000, 40, FP64, (49,)),
]


@pytest.mark.parametrize("nr,nz,rb,good", RZ)
def test_rows_of_the_rz_chunks(nr, nz, rb, good):
    strips = (nz + 1 + 55) // 56
    assert host_plan.lib().rz_rows(nr + 1, strips, rb == FP32) in good
    assert host_plan.lib().rz_rows(nr + 1, 1, rb == FP32) >= 12


def test_rows_of_the_rz_chunks_from_all_counts():
    """The counts of chunks passed over have the rows of one that is tried."""
    def every(nr1, nzt, fp32):
        best = None
        for chunks in range(1, (nr1 + 11) // 12 + 1):
            rows = max(12, -(-nr1 // chunks))
            n = -(-nzt * -(-nr1 // rows) // 1024)
            cost = (rows + 16) * (max(3, n) if fp32 else (n + 1) // 2 * 2)
            if best is None or cost < best[0]:
                best = (cost, rows)
        return best[1]
    for nr1 in (3, 11, 12, 13, 24, 25, 100, 301, 1001, 1777, 20011):
        for nzt in (1, 2, 17, 82, 325, 1200):
            for fp32 in (False, True):
                assert host_plan.lib().rz_rows(nr1, nzt, fp32) == every(nr1, nzt, fp32), (nr1, nzt, fp32)


def test_rows_of_the_rz_energy():
    """No march longer than needed to give each of 8192 waves an item."""
    f = host_plan.lib().rz_energy
    assert f(25, 5) == f(301, 5) == f(61, 11) == 1
    assert f(1001, 285) == 16 and f(100001, 1) == 12
    for nr1 in (3, 100, 5000, 10 ** 6):
        for nzt in (1, 7, 300):
            rows = f(nr1, nzt)
            assert 1 <= rows <= 16 and (rows == 1 or nzt * -(-nr1 // rows) >= 8192)


def _every_plan(tiles, nplanes, xmax, fill, unroll, tail):
    """The plan of the chunks from every count of them in turn."""
    planes = lambda xc: float(-(-(xc + fill) // unroll) * unroll)
    best = None
    for nxc in range(-(-nplanes // xmax), nplanes + 1):
        xc = -(-nplanes // nxc)
        if -(-nplanes // xc) != nxc:
            continue
        items = tiles * nxc
        if (best and items > 32 * 256) or items > 0x3fffffff:
            break
        rem = items % 256
        p = (xc, nxc, items, items, 1, xc)
        rounds = -(-items // 256) * planes(xc)
        if tail and rem and items > 256:
            base = items // 256 * planes(xc)
            for s in range(2, min(256 // rem, xc) + 1):
                tc = -(-xc // s)
                if base + planes(tc) < rounds:
                    rounds = base + planes(tc)
                    split = -(-xc // tc)
                    p = (xc, nxc, items - rem, items - rem + rem * split, split, tc)
        cost = rounds + 0.25 * items * planes(xc) / 256
        if best is None or cost < best[0]:
            best = (cost, p)
    return best[1]


def test_chunk_plans_from_all_counts():
    for tiles in (1, 2, 6, 35, 117, 257, 468, 1820):
        for nplanes in (2, 3, 25, 97, 129, 513, 1001, 1777):
            for xmax in (1, 5, 31, 64, 1 << 20):
                for fill, unroll, tail in ((10, 1, 1), (2, 3, 0)):
                    a = (tiles, nplanes, xmax, fill, unroll, tail)
                    assert host_plan.plan(*a) == _every_plan(*a), a


def test_chunk_plans_cost_no_launch():
    """A plan is made for every launch: on a long thin grid it may not try every
    count of chunks (77 us on one tile of 16001 planes)."""
    best = 1.0
    for _ in range(30):
        t = time.perf_counter()
        for _ in range(10):
            host_plan.plan(1, 16001, 1 << 20, 10, 1, 1)
        best = min(best, (time.perf_counter() - t) / 10)
    assert best < 40e-6, best


def test_batch_chunks():
    # one member that fits a round in two chunks is not cut to 48 planes
    assert host_plan.batch([(117, 129)], 256, 48, 10) == (65, True)
    # few tiles: chunks short enough to give every workgroup an item
    c, one = host_plan.batch([(4, 30), (5, 41), (3, 26)], 256, 48, 10)
    assert one and c <= 3
    # many rounds: the longest chunks allowed, or nearly
    c, one = host_plan.batch([(100, 129)] * 64, 256, 24, 10)
    assert not one and 20 <= c <= 24
    # single steps of a member longer than a chunk's limit
    c, one = host_plan.batch([(81, 161)] * 8, 256, 24, 6)
    assert not one and c <= 24


def test_batch_chunks_are_the_shortest_in_all():
    rng = random.Random(5)
    for _ in range(200):
        n, grid, cap, fill = rng.randint(1, 12), rng.choice((32, 256)), rng.choice((24, 48)), rng.choice((6, 10))
        m = [(rng.choice((1, 4, 20, 117, 300)), rng.randint(2, 200)) for _ in range(n)]
        c, one = host_plan.batch(m, grid, cap, fill)
        items = lambda c: sum(t * -(-p // c) for t, p in m)
        rounds = lambda c: max(1, -(-items(c) // grid))
        assert 1 <= c <= max(p for _, p in m) and one == (items(c) <= grid) and (one or c <= cap), (m, c)
        # no other chunk of as many rounds, or of up to three more, takes less
        allowed = [q for q in range(1, max(p for _, p in m) + 1) if q <= cap or items(q) <= grid]
        near = [q for q in allowed if rounds(q) <= rounds(min(max(allowed), cap)) + 3 or rounds(q) == 1]
        assert rounds(c) * (c + fill) <= min(rounds(q) * (q + fill) for q in near), (m, c)


def _active_count(on, xc):
    planes = on.shape[0]
    return sum(int(on[max(0, xs - 4):min(xs + xc, planes) + 4].any(axis=0).sum()) for xs in range(0, planes, xc))


# tiles on along a pipe with a wide entrance and exit and a narrow middle, over the
# planes across it: the 512 x 512 x 2048 taper in tiles of 10 rows by 28 and 60
# entries, a small one, and grids wholly on and off
@pytest.mark.parametrize("planes,nyt,nzt,wide", [(513, 52, 74, 0.25), (513, 52, 35, 0.25), (97, 10, 9, 0.3), (201, 21, 15, 0.25),
                                                 (129, 13, 18, 2.0), (129, 13, 18, 0.0), (41, 1, 1, 2.0)])
def test_chunk_of_the_active_tiles(planes, nyt, nzt, wide):
    x = (np.arange(planes) + 0.5) / planes - 0.5
    y = (np.arange(nyt) + 0.5) / nyt - 0.5
    z = np.abs((np.arange(nzt) + 0.5) / nzt - 0.5)
    r = np.minimum(0.2 * wide + 1.5 * wide * z, wide)
    on = (x[:, None, None] ** 2 + y[None, :, None] ** 2 < (r * r)[None, None, :]).reshape(planes, -1)
    cost = {}
    for c in range(1, planes + 1):
        xc = -(-planes // c)
        if -(-planes // xc) != c or xc in cost or (xc < 24 and c * on.shape[1] > 20000):
            continue
        items = _active_count(on, xc)
        cost[xc] = (-(-items // 256) + 0.25 * items / 256) * (xc + 10)
    got = host_plan.active(on, 1 << 30)
    assert got in cost
    # within 5 % of the least over all chunks of at least 24 planes, or of any that fill a round
    assert cost[got] <= 1.05 * min(v for k, v in cost.items() if k >= 24 or v < 4 * 40)
    assert host_plan.active(on, 30) <= 30
