"""Large batches in two tails: the results of a handle's plain, timed, pipelined
and projection runs and of the single call, with a register class and with the
pairs above the classes in the first tail.  Every result is checked at a random
point modulo a 61-bit prime against the determinant there.
"""
import random

import numpy as np
import pytest

import paper_1103_4697_amd as snc
import synth
from oracle import resultant as R
from oracle import zx

pytestmark = pytest.mark.gpu

Q61 = (1 << 61) - 1


def _dense(rnd, m, dx, bits):
    return [[rnd.randrange(-(1 << bits) + 1, 1 << bits) for _ in range(dx)] + [rnd.randrange(1, 1 << bits)]
            for _ in range(m + 1)]


def _class_first(rnd):
    pairs = [(_dense(rnd, 1, 600, 1500), _dense(rnd, 1, 600, 1500)) for _ in range(11)]
    for i in range(9):  # the classes alternate, so the tails reorder the batch
        pairs.insert(2 * i, (_dense(rnd, 20, 20, 60), _dense(rnd, 19, 20, 60)))
    return pairs


def _general_first(rnd):
    pairs = [(_dense(rnd, 70, 8, 64), _dense(rnd, 69, 8, 64)) for _ in range(4)]
    pairs += [(_dense(rnd, 60, 20, 24), _dense(rnd, 59, 20, 24)) for _ in range(4)]
    pairs.insert(1, (_dense(rnd, 4, 4, 12), _dense(rnd, 3, 4, 12)))
    pairs.insert(3, ([[1, 2], [3, 4]], []))  # a trivial one
    return pairs


def _check(pairs, got, rnd):
    assert len(got) == len(pairs)
    for i, ((f, g), r) in enumerate(zip(pairs, got)):
        if not f or not g:
            assert r == []
            continue
        x0 = rnd.randrange(Q61)
        assert zx.evaluate(r, x0) % Q61 == R.resultant_at_mod(f, g, x0, Q61), f"pair {i}"


@pytest.mark.parametrize("make", [_class_first, _general_first])
def test_every_kind_of_run(make, assert_same):
    rnd = random.Random(31)
    pairs = make(rnd)
    plans = [snc.resultant_plan(f, g) for f, g in pairs]
    assert sum((p.deg_bound + 1) * p.out_nlimbs for p in plans) >= 1 << 20  # large enough for two tails
    ctx = snc.Context(0)
    b = snc.ResultantBatch(pairs, ctx)
    b.run()
    want = b.results()
    _check(pairs, want, rnd)
    b.run()  # replays
    assert_same(b.results(), want, "second run")
    t0 = b.submit()
    b.run()  # beside an outstanding run
    assert_same(b.results(), want, "run beside a submitted one")
    t1 = b.submit()
    b.collect(t0)
    assert_same(b.results(), want, "first submitted run")
    b.collect(t1)
    assert_same(b.results(), want, "second submitted run")
    ctx.set_timing(True)
    b.run()
    ctx.set_timing(False)
    assert_same(b.results(), want, "timed run")
    b.run()
    assert_same(b.results(), want, "run after the timed one")
    b.close()
    assert_same(snc.resultant_y_batch(pairs, ctx), want, "single call")
    small = [([[1, 2], [3, 4]], [[5, 6], [7, 8]])]
    for r, (f, g) in zip(snc.resultant_y_batch(small, ctx), small):  # the staging blocks again, with a small call
        assert r == R.resultant_y(f, g)


def test_projection_run():
    """run_sqfree takes all jobs in one tail: gcd(R, R') of random pairs is 1."""
    rnd = random.Random(32)
    pairs = _class_first(rnd)
    b = snc.ResultantBatch(pairs, snc.Context(0))
    b.run()
    want = b.results()
    b.run_sqfree()
    assert b.results() == want
    assert all(g == [1] for g in b.sqfree_results())
    b.run()
    assert b.results() == want


def test_every_pair_of_a_grouped_batch():
    """More than 4,096 (pair, prime) instances of degree bounds 63 to 1600, jobs sharing interpolation workgroups."""
    rng = np.random.default_rng(8821)
    shapes = [(7, 9, 12, 12), (8, 8, 16, 16), (9, 7, 20, 8), (16, 8, 30, 30), (31, 33, 24, 24), (40, 40, 32, 32)]
    pairs = [synth.random_pair(rng, *sh) for sh in shapes]
    while sum(snc.resultant_plan(f, g).nprimes for f, g in pairs) < 4300:
        df, dg = int(rng.integers(8, 41)), int(rng.integers(8, 41))
        pairs.append(synth.random_pair(rng, df, dg, int(rng.integers(8, 33)), int(rng.integers(8, 33))))
    pairs = [([[int(c) for c in r] for r in f], [[int(c) for c in r] for r in g]) for f, g in pairs]
    _check(pairs, snc.resultant_y_batch(pairs), random.Random(8822))
