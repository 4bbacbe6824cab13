"""Short quotients of the modular gcd's exact divisions: the power series of
1 / G stops at the longer quotient's length and the last block's products at
its own, so lengths on the edges of sixteen, for quotients of equal and of
different lengths, and dividends whose degree drops mod the first prime."""
import random

import pytest

import paper_1103_4697_amd as snc
import synth

pytestmark = pytest.mark.gpu


def _poly(rnd, deg, lead):
    return [rnd.randint(-99, 99) for _ in range(deg)] + [lead]


@pytest.mark.parametrize("e", [1, 3, 20, 70])
@pytest.mark.parametrize("du,dv", [(0, 0), (1, 1), (2, 1), (14, 0), (15, 14), (16, 15), (17, 31), (32, 33), (47, 48), (63, 2),
                                   (1, 64), (79, 80)])
def test_planted_factor(e, du, dv):
    rnd = random.Random(1000 * e + du)
    h = _poly(rnd, e, 1)
    u, v = _poly(rnd, du, 3), _poly(rnd, dv, 2)
    assert snc.gcd_z(synth.univariate_product(h, u), synth.univariate_product(h, v)) == h


@pytest.mark.parametrize("first", [True, False])
@pytest.mark.parametrize("e,du", [(2, 1), (9, 16), (30, 33)])
def test_leading_coefficient_vanishing_mod_a_prime(first, e, du):
    rnd = random.Random(e + du)
    h = _poly(rnd, e, 1)
    a = synth.univariate_product(h, _poly(rnd, du, snc.prime(0)))
    b = synth.univariate_product(h, _poly(rnd, du, 7))
    assert snc.gcd_z(*((a, b) if first else (b, a))) == h
