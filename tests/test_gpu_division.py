"""The modular gcd's exact divisions by the monic gcd, 64 quotient
coefficients at a time: gcd degrees and quotient lengths on the block edges
and over the register classes.  The result is certified from the lifted
cofactors, so a wrong quotient coefficient cannot give the planted factor."""
import random

import pytest

import paper_1103_4697_amd as snc
import synth

pytestmark = pytest.mark.gpu


def _poly(rnd, deg, lead=None):
    return [rnd.randint(-99, 99) for _ in range(deg)] + [lead or rnd.choice([1, 2, 3, 5])]


@pytest.mark.parametrize("e", [1, 2, 15, 16, 17, 63, 64, 65, 127, 130])
@pytest.mark.parametrize("du,dv", [(1, 0), (62, 63), (64, 65), (129, 1), (300, 257)])
def test_planted_factor(e, du, dv):
    rnd = random.Random(1000 * e + du)
    h = _poly(rnd, e, 1)
    u, v = _poly(rnd, du, 3), _poly(rnd, dv, 2)
    a, b = synth.univariate_product(h, u), synth.univariate_product(h, v)
    got = snc.gcd_z(a, b)
    # h divides the gcd; a factor that the random u and v share would show as a larger degree
    assert got == h


@pytest.mark.parametrize("e,du", [(40, 200), (64, 63)])
def test_leading_coefficient_vanishing_mod_a_prime(e, du):
    """a's leading coefficient is divisible by the first table prime: the dividend's degree drops mod it."""
    rnd = random.Random(e + du)
    h = _poly(rnd, e, 1)
    u, v = _poly(rnd, du, snc.prime(0)), _poly(rnd, du - 3, 7)
    assert snc.gcd_z(synth.univariate_product(h, u), synth.univariate_product(h, v)) == h


@pytest.mark.parametrize("degs", [(33, 1), (64, 31), (100, 65)])
def test_quotients_in_the_square_free_factorisation(degs):
    rnd = random.Random(sum(degs))
    f1, f2 = _poly(rnd, degs[0], 1), _poly(rnd, degs[1], 1)
    a = [4 * c for c in synth.univariate_product(f1, synth.univariate_product(f2, f2))]
    assert snc.sqfree_factor(a) == (4, [(f1, 1), (f2, 2)])
