"""Interpolation on the matrix cores: degree bounds on the edges of its
64-point blocks and 16-row tiles and of its one-order/two-order line, and
groups of jobs with different prime counts.

Pairs linear in y have the resultant a1 b0 - a0 b1, so the integer result is
exact plain Python.
"""
import random

import numpy as np
import pytest

import paper_1103_4697_amd as snc

pytestmark = pytest.mark.gpu


def _pair(rnd, d1, d2, bits):
    """f, g linear in y with coefficients of up to `bits` bits and deg_x d1, d2: degree bound d1 + d2."""
    def row(d):
        return [rnd.getrandbits(bits) - (1 << (bits - 1)) for _ in range(d)] + [(1 << (bits - 1)) - 1]
    return [row(d1), row(d1)], [row(d2), row(d2)]


def _want(f, g):
    def mul(a, b):
        return np.convolve(np.array(a, dtype=object), np.array(b, dtype=object))
    r = [int(v) for v in mul(f[1], g[0]) - mul(f[0], g[1])]
    while r and r[-1] == 0:
        r.pop()
    return r


@pytest.mark.parametrize("n1", [1, 2, 63, 64, 65, 127, 128, 129, 130, 255, 257, 1024, 1025, 2047, 2049, 4097, 8191, 8193])
def test_block_and_tile_edges(n1):
    rnd = random.Random(n1)
    D = n1 - 1
    f, g = _pair(rnd, D // 2, D - D // 2, 12)
    assert snc.resultant_plan(f, g).deg_bound == D
    assert snc.resultant_y(f, g) == _want(f, g)


@pytest.mark.parametrize("njobs,bits", [(23, 2000), (19, 13500)])
def test_groups_of_jobs(njobs, bits):
    """Enough (resultant, prime) pairs that jobs share workgroups, with prime counts and degrees that differ
    inside a group; replays of the graph."""
    rnd = random.Random(njobs)
    pairs = []
    for i in range(njobs):
        d1, d2 = rnd.randint(0, 70), rnd.randint(1, 70)
        pairs.append(_pair(rnd, d1, d2, bits - 37 * i))
    ks = [snc.resultant_plan(f, g).nprimes for f, g in pairs]
    assert sum(ks) >= 2048 and len(set(ks)) > 3
    want = [_want(f, g) for f, g in pairs]
    b = snc.ResultantBatch(pairs)
    for _ in range(3):
        b.run()
        assert b.results() == want


@pytest.mark.parametrize("d", [4, 20, 64])
@pytest.mark.parametrize("roots", [1, 3, 40])
def test_abnormal_points_beside_normal_ones(d, roots):
    """lc_y(f) vanishes at the first `roots` evaluation points of the first prime's power sequence
    (1, q, q^2, .. as integers: q is 2 or 3 for every prime of the table's head), so some points of a prime
    take the general elimination and the others do not; against y-reversed operands, whose leading
    coefficients are constants: res(y^m f(1/y), y^n g(1/y)) = (-1)^(mn) res(f, g)."""
    rnd = random.Random(100 * d + roots)
    lc = [1]
    for i in range(min(roots, 12)):  # (x - 2^i): integer roots shared by every prime
        lc = [int(v) for v in np.convolve(np.array(lc, dtype=object), np.array([-(2 ** i), 1], dtype=object))]
    m, n = d, max(d - 1, 1)
    f = [[rnd.randint(1, 99)]] + [[rnd.randint(-99, 99), rnd.randint(-9, 9)] for _ in range(m - 1)] + [lc]
    g = [[rnd.randint(1, 99)]] + [[rnd.randint(-99, 99)] for _ in range(n - 1)] + [[rnd.randint(1, 99)]]
    got = snc.resultant_y(f, g)
    rev = snc.resultant_y(f[::-1], g[::-1])
    assert got == [(-1) ** (m * n) * c for c in rev]
    assert got
