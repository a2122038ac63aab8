"""The anchored sums of the real path's lanes (GPU): leaves whose terms spread
too far for the first anchor, or for any, run again and give the same exact
sums; terms below 1 and of any order are summed as well."""
import sys

import numpy as np
import pytest

import bounds
from oracle import oracle as orc
from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    from paper_2109_04528_amd import Context
    c = Context()
    yield c
    c.close()


def product(x, seed):
    """Product state whose mode i multiplies a term by x[i] when it is in the subset."""
    # x = 1 / sqrt(det of the block), a pure squeezed vacuum: x = cosh r
    r = np.arccosh(np.asarray(x, dtype=np.float64))
    rng = np.random.default_rng(seed)
    return gen.product_state_O(r, 1.0, rng.uniform(0.0, 2.0 * np.pi, r.size))


# spread of a leaf's terms 2^(11 log2 x): 2^11 (well inside the first anchor's
# 2^30), 2^29 to 2^31 (about it), 2^40 (raised once or twice), all below 2^53 in total
@pytest.mark.parametrize("n", [12, 14, 18])
@pytest.mark.parametrize("lg", [1.0, 2.6, 2.7, 2.75, 2.8, 2.9])
def test_whole_state_equals_the_stored_terms_sum(ctx, n, lg):
    # the first modes stay dim so that the whole sum stays exact; the last 11 spread
    x = np.concatenate([np.full(n - 11, 1.1), np.full(11, 2.0 ** lg)])
    O = product(x, n)
    r = ctx.eval(O)
    _, _, w = ctx.click_all(O)  # every term stored, then summed exactly
    say(f"case anchor n={n} spread 2^{11 * lg:.0f}: {r.tor!r} closed form {np.prod(x - 1.0)!r}")
    assert r.path == 1 and r.status == 0
    assert (r.tor, r.tor_lo) == (w.tor, w.tor_lo)
    assert abs(r.sum_abs - w.sum_abs) <= 1e-12 * w.sum_abs


# beyond every anchor: the sums are double-double as before
@pytest.mark.parametrize("n", [11, 13, 16])
@pytest.mark.parametrize("lg", [4.6, 6.0])
def test_spread_beyond_every_anchor(ctx, n, lg):
    x = np.full(n, 2.0 ** lg)
    r = ctx.eval(product(x, n))
    want, tot = np.prod(x - 1.0), np.prod(x + 1.0)
    # each term's relative error: a few units per mode, conditioned by the block
    tol = 8 * n * 2.0 ** -53 * 2.0 ** (2 * lg) * tot
    say(f"case anchor beyond n={n} lg={lg}: rel={abs(r.value - want) / want:.2e}")
    assert r.status == 0 and tol <= 1e-2 * want and abs(r.value - want) <= tol


@pytest.mark.parametrize("n", [6, 11, 13, 15])
@pytest.mark.parametrize("c,shift", [(-0.5, 0.0), (0.5, 3.0), (0.5, 30.0)])
def test_terms_below_one(ctx, n, c, shift):
    """I - O with eigenvalues above 1 (about 1, 4 and 31): terms below 1, a
    subset's the smaller the more modes it has."""
    O = c * gen.structured_O(gen.random_O(n, 60 + n, 0.5, 1.2, 0.9)) - shift * np.eye(2 * n)
    r = ctx.eval(O)
    want = orc.tor(O, mode=orc.QUAD, threads=8)
    tol = bounds.sum_bound(want.sum_sq, bounds.U64, bounds.UNIT_OF_MODE["quad"])
    say(f"case anchor below one n={n} c={c} shift={shift}: rel={abs(r.value - want.value) / abs(want.value):.2e} tol={tol / abs(want.value):.2e}")
    assert r.path == 1 and r.status == 0 and abs(r.value - want.value) <= tol
    assert abs(r.sum_abs - want.sum_abs) <= 1e-12 * want.sum_abs
