"""The queue of subtree roots (GPU): a wave's first root is its own block's,
the later ones come from the counter.  Launches of fewer, as many and more
roots than waves, alone and in ragged batches, give every root the same
partial whatever wave runs it, so the result does not depend on the number of
waves, bit for bit."""
import sys

import numpy as np
import pytest

from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def bits(r):
    return (r.tor, r.tor_lo, r.sum_abs, r.status, r.path)


@pytest.mark.parametrize("form", ["real", "hermitian", "dd"])
@pytest.mark.parametrize("k", [7, 8, 9])  # 128, 256 and 512 roots for 256 waves (one per CU)
def test_roots_against_waves(form, k):
    from paper_2109_04528_amd import Context, TOR_FACTOR_DD
    flags = TOR_FACTOR_DD if form == "dd" else 0
    # one mode below the split, several, and a matrix smaller than the leaf
    mats = [(gen.random_hpd_O if form == "hermitian" else gen.random_O)(n, 70 + n) for n in (21, 20, 18, 5)]
    with Context(device=0, flags=flags, split_k=k, waves_per_cu=1) as one, \
            Context(device=0, flags=flags, split_k=k) as full:
        for O in mats:
            say(f"case queue {form} k={k} n={O.shape[0] // 2}")
            a, b = one.eval(O), full.eval(O)
            assert a.status == 0 and bits(a) == bits(b)
        say(f"case queue {form} k={k} batch")
        for a, b in zip(one.eval_batch(mats + mats[::-1]), full.eval_batch(mats + mats[::-1])):
            assert a.status == 0 and bits(a) == bits(b)


def test_single_root_matrices_in_one_launch():
    from paper_2109_04528_amd import Context
    # 300 queue items of one root each for 256 waves: 44 come from the counter
    mats = [gen.random_O(1 + i % 11, i) for i in range(300)]
    say("case queue 300 single-root matrices")
    with Context(device=0, waves_per_cu=1, split_k=1) as ctx, Context(device=0) as ref:
        got = ctx.eval_batch(mats)
        for i in range(0, 300, 23):
            assert bits(got[i]) == bits(ref.eval(mats[i]))
        assert np.all([r.status == 0 for r in got])


# subsets per wave from 2^1 to 2^15: roots of one leaf, of a few, several per wave
@pytest.mark.parametrize("form", ["real", "hermitian", "dd"])
@pytest.mark.parametrize("sizes", [(11, 3), (14, 15, 16), (18,) * 12, (20, 17, 12, 9, 19), (21, 22, 16), (23, 10, 22)])
def test_batch_split_does_not_change_values(form, sizes):
    from paper_2109_04528_amd import Context, TOR_FACTOR_DD
    make = gen.random_hpd_O if form == "hermitian" else gen.random_O
    mats = [make(n, 500 + 7 * i + n) for i, n in enumerate(sizes)]
    say(f"case batch split {form} {sizes}")
    with Context(flags=TOR_FACTOR_DD if form == "dd" else 0) as ctx:
        for O, r in zip(mats, ctx.eval_batch(mats)):
            lone = ctx.eval(O)
            assert r.status == 0 and r.path == lone.path
            if form == "real":  # exact sums of the same terms
                assert (r.tor, r.tor_lo) == (lone.tor, lone.tor_lo)
            else:  # the same terms, double-double sums of another grouping
                assert abs((r.tor - lone.tor) + (r.tor_lo - lone.tor_lo)) <= 2.0 ** -90 * lone.sum_abs
