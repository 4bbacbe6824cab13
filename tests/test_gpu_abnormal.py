"""Points at which the elimination's regular schedule fails: the general
elimination inside the interpolation, a wavefront or a pair of lanes each.

Expected values are plain integer polynomials: res_y(F(y^g), G(y^g)) =
res_y(F, G)^g, whose remainders skip degrees at every point (linear F and G:
(a1 b0 - a0 b1)^g), and res_y(f, b1 y + b0) = (-1)^m sum_i f_i (-b0)^i b1^(m-i)
with lc_y(f) planted to vanish modulo the first prime at chosen evaluation
points.
"""
import random
import time

import numpy as np
import pytest

import paper_1103_4697_amd as snc

pytestmark = pytest.mark.gpu


def _mul(a, b):
    return [int(v) for v in np.convolve(np.array(a, dtype=object), np.array(b, dtype=object))]


def _sub(a, b):
    n = max(len(a), len(b))
    a, b = a + [0] * (n - len(a)), b + [0] * (n - len(b))
    return [x - y for x, y in zip(a, b)]


def _trim(a):
    while a and a[-1] == 0:
        a.pop()
    return a


def _poly(rnd, d, bits):
    return [rnd.randrange(-(1 << bits) + 1, 1 << bits) for _ in range(d)] + [rnd.randrange(1, 1 << bits)]


def _power_pair(rnd, g, d1, d2, bits):
    """f = a1 y^g + a0, g = b1 y^g + b0 and their resultant."""
    a1, a0 = _poly(rnd, d1, bits), _poly(rnd, d1, bits)
    b1, b0 = _poly(rnd, d2, bits), _poly(rnd, d2, bits)
    r, base = [1], _sub(_mul(a1, b0), _mul(a0, b1))
    for _ in range(g):
        r = _mul(r, base)
    zero = [[0]] * (g - 1)
    return [a0] + zero + [a1], [b0] + zero + [b1], _trim(r)


def _points(n):
    """The evaluation points q^i, -q^i of the first prime, in order."""
    p = snc.prime(0)
    q = 1
    while True:
        q += 1
        t, ok = 1, True
        for _ in range(5000):
            t = t * q * q % p
            if t == 1:
                ok = False
                break
        if ok:
            break
    return [s * pow(q, i, p) % p for i in range((n + 1) // 2) for s in (1, -1)][:n]


def _linear_divisor_pair(rnd, m, roots, d):
    """f of y-degree m whose leading coefficient vanishes at `roots` modulo the first prime, and a divisor linear
    in y, with their resultant."""
    p = snc.prime(0)
    lc = [1]
    for x in roots:
        lc = [v % p for v in _mul(lc, [-x, 1])]
    f = [_poly(rnd, d, 6) for _ in range(m)] + [lc]
    b1, b0 = _poly(rnd, d, 5), _poly(rnd, d, 5)
    acc, mb0 = [0], [-v for v in b0]
    power = [1]
    for row in reversed(f):  # Horner in -b0 / b1
        acc = _sub(_mul(acc, mb0), [-v for v in _mul(row, power)])
        power = _mul(power, b1)
    return f, [b0, b1], _trim([(-1) ** m * v for v in acc])


@pytest.mark.parametrize("g,dx", [(2, 1), (2, 63), (2, 64), (2, 150), (3, 3), (4, 0), (4, 7), (4, 40), (16, 2), (16, 11),
                                  (17, 12), (33, 3), (40, 4), (63, 1), (64, 2)])
def test_every_point(g, dx):
    rnd = random.Random(100 * g + dx)
    f, h, want = _power_pair(rnd, g, dx, dx + 1, 9)
    assert snc.resultant_y(f, h) == want


@pytest.mark.parametrize("rows", [4, 5, 8, 9, 12, 13, 16, 17])
def test_every_point_row_lengths(rows):
    """Rows of all lengths modulo a pair of chunks, two nonzero rows per operand in groups of their own."""
    rnd = random.Random(rows)
    f, h, want = _power_pair(rnd, 6, rows - 1, rows // 2, 20)
    assert snc.resultant_y(f, h) == want


@pytest.mark.parametrize("m", [2, 15, 16, 33, 64])
@pytest.mark.parametrize("marks", [1, 8, 9, 32, 33, 100])
def test_some_points(m, marks):
    """One mark to more than a workgroup gives its wavefronts, at y-degrees on both sides of 16."""
    rnd = random.Random(1000 * m + marks)
    roots = _points(marks) if marks % 2 else _points(2 * marks)[1::2]  # pairs, or one point of each pair
    f, h, want = _linear_divisor_pair(rnd, m, roots, max(3, marks // m + 1))
    assert snc.resultant_plan(f, h).deg_bound + 1 >= 2 * marks or marks % 2
    assert snc.resultant_y(f, h) == want


def test_marks_of_jobs_that_share_workgroups():
    """Pairs with every, with some and without abnormal points, of y-degrees below and above 16, in groups."""
    rnd = random.Random(77)
    items = []
    for i in range(8):
        items.append(_power_pair(rnd, 2 + i % 3, 3 + i, 2, 500 + 11 * i))
        items.append(_power_pair(rnd, 17 + i, 1, 1, 60))
        items.append(_linear_divisor_pair(rnd, 20 if i % 2 else 3, _points(3 + 9 * i), 4))
        items.append(_power_pair(rnd, 1, 30 + i, 25, 1500 + 37 * i))
    pairs = [(f, h) for f, h, _ in items]
    want = [w for _, _, w in items]
    assert sum(snc.resultant_plan(f, h).nprimes for f, h in pairs) >= 2 * 1024  # jobs share workgroups from here
    b = snc.ResultantBatch(pairs)
    for _ in range(3):
        b.run()
        assert b.results() == want


def _best(f, n=5):
    f()
    t = []
    for _ in range(n):
        t0 = time.perf_counter()
        f()
        t.append(time.perf_counter() - t0)
    return min(t)


def test_every_point_beside_the_dense_pair():
    """The general elimination keeps within a factor of the regular one: y-degree 4, x-degree 700, even in y
    against dense.  One lane after the other through dependent loads took 60 times the dense pair."""
    rnd = random.Random(9)

    def rows(step):
        return [_poly(rnd, 700, 7) if i % step == 0 else [0] for i in range(5)]
    even, dense = snc.ResultantBatch([(rows(2), rows(2))]), snc.ResultantBatch([(rows(1), rows(1))])
    te, td = _best(even.run), _best(dense.run)
    print(f"even {te * 1e6:.0f} us, dense {td * 1e6:.0f} us")
    assert te < 20 * td
