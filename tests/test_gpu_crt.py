"""Chinese remaindering on the matrix cores (more than 64 primes).

Pairs linear in y have the resultant a1 b0 - a0 b1 in closed form, so the
integer result is exact plain Python at any coefficient size; the sizes put
the number of primes on the edges of the 64-prime blocks, of the two row
variants of the digits kernel and of the whole table, and the number of
coefficients on the edges of its tiles.
"""
import random

import pytest

import paper_1103_4697_amd as snc

pytestmark = pytest.mark.gpu


def _pair(k, dx, seed, extreme=False):
    """f = a1 y + a0, g = b1 y + b0 with deg_x = dx whose plan takes exactly k primes."""
    rnd = random.Random(seed)
    bits = 15 * k - 8

    def coef(b):
        v = (1 << b) - 1 if extreme else rnd.getrandbits(b) | (1 << (b - 1))
        return v

    for _ in range(400):
        a1, a0, b1 = ([coef(bits) * (1 if extreme else rnd.choice((-1, 1))) for _ in range(dx + 1)] for _ in range(3))
        b0 = [coef(bits) * (1 if extreme else rnd.choice((-1, 1))) for _ in range(dx + 1)]
        if extreme:
            b1 = [-c for c in b1]
        f, g = [a0, a1], [b0, b1]
        got = snc.resultant_plan(f, g).nprimes
        if got == k:
            return f, g
        bits += 7 * (k - got) if abs(k - got) > 1 else (k - got) * 3
    raise AssertionError(f"no coefficient size takes {k} primes")


def _want(f, g):
    def mul(a, b):
        c = [0] * (len(a) + len(b) - 1)
        for i, x in enumerate(a):
            for j, y in enumerate(b):
                c[i + j] += x * y
        return c
    r = [x - y for x, y in zip(mul(f[1], g[0]), mul(f[0], g[1]))]
    while r and r[-1] == 0:
        r.pop()
    return r


@pytest.mark.parametrize("k,dx", [(64, 3), (65, 4), (66, 8), (127, 3), (128, 7), (129, 32), (192, 2), (193, 12),
                                  (517, 40), (2240, 1), (2241, 4), (3072, 2)])
def test_linear_pair(k, dx):
    f, g = _pair(k, dx, 7 * k + dx)
    assert snc.resultant_y(f, g) == _want(f, g)


@pytest.mark.parametrize("k", [65, 128, 129, 448, 2241])
@pytest.mark.parametrize("sign", [1, -1])
def test_largest_values_of_both_signs(k, sign):
    """Constant coefficients with every product of one sign: the result attains the coefficient bound."""
    f, g = _pair(k, 0, k, extreme=True)
    g = [[sign * c for c in row] for row in g]
    got = snc.resultant_y(f, g)
    assert got == _want(f, g)
    assert got[0] * sign > 0


def test_mixed_sizes_in_one_batch():
    """Jobs on both sides of the 64-prime line and of the tile edges in one launch, graph replayed."""
    pairs = [_pair(k, dx, 100 * k + dx) for k, dx in [(3, 5), (64, 7), (65, 7), (97, 8), (130, 3), (200, 0), (321, 31)]]
    want = [_want(f, g) for f, g in pairs]
    b = snc.ResultantBatch(pairs)
    for _ in range(3):
        b.run()
        assert b.results() == want


@pytest.mark.parametrize("nl", [1, 2, 3, 4, 5, 63, 64, 65, 128, 130])
@pytest.mark.parametrize("dx", [2, 300])
def test_input_reduction_limb_edges(nl, dx):
    """Coefficients on the limb edges of both signs, reduced inside the evaluation (small degree) and, with
    many coefficients, points and primes, by the launch before it."""
    rnd = random.Random(1000 * nl + dx)
    top = 32 * nl - 1
    edges = [0, 1, -1, (1 << top) - 1, -(1 << top), 1 << (32 * (nl // 2)), -(1 << (32 * (nl // 2))),
             (1 << (32 * (nl // 2))) - 1 if nl > 1 else 7]

    def row():
        return [rnd.choice(edges) if rnd.random() < 0.7 else rnd.getrandbits(top) for _ in range(dx)] + [-(1 << top)]
    f, g = [row(), row()], [row(), row()]
    assert snc.resultant_y(f, g) == _want(f, g)
