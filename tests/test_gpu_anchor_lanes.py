"""The anchors of the real path's sums are each lane's own (GPU): states whose
last five modes, a lane's share, spread its terms to below, about and beyond
the first anchor, and beyond all of them, where the leaves of a root run
without."""
import sys

import numpy as np
import pytest

from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def product(x, seed):
    """Product state whose mode i multiplies a term by x[i] when it is in the subset."""
    r = np.arccosh(np.asarray(x, dtype=np.float64))
    rng = np.random.default_rng(seed)
    return gen.product_state_O(r, 1.0, rng.uniform(0.0, 2.0 * np.pi, r.size))


# spread of a lane's terms 2^(5 lg): 2^20, 2^33 to 2^35 (about the first anchor), 2^39, 2^43
@pytest.mark.parametrize("n,split_k", [(11, 0), (13, 0), (13, 1)])
@pytest.mark.parametrize("lg", [4.0, 6.6, 6.8, 7.0, 7.8, 8.6])
def test_whole_state_equals_the_stored_terms_sum(n, split_k, lg):
    from paper_2109_04528_amd import Context
    # the others stay dim so that the whole sum stays below 2^53 and exact
    O = product(np.concatenate([np.full(n - 5, 1.1), np.full(5, 2.0 ** lg)]), n)
    with Context(split_k=split_k) as ctx:
        r = ctx.eval(O)
        _, _, w = ctx.click_all(O)
    say(f"case lane anchor n={n} k={split_k} spread 2^{5 * lg:.0f}: {r.tor!r}")
    assert r.path == 1 and r.status == 0
    assert (r.tor, r.tor_lo) == (w.tor, w.tor_lo)
    assert abs(r.sum_abs - w.sum_abs) <= 1e-12 * w.sum_abs


# 2^52 and 2^60 a lane: four leaves of a root raise the anchors, the rest run without
@pytest.mark.parametrize("n,split_k", [(11, 0), (16, 1), (16, 5)])
@pytest.mark.parametrize("lg", [10.4, 12.0])
def test_spread_beyond_every_anchor(n, split_k, lg):
    from paper_2109_04528_amd import Context
    x = np.concatenate([np.full(n - 5, 4.0), np.full(5, 2.0 ** lg)])
    with Context(split_k=split_k) as ctx:
        r = ctx.eval(product(x, n))
    want, tot = np.prod(x - 1.0), np.prod(x + 1.0)
    # each term's relative error: a few units per mode, conditioned by the block
    tol = 8 * n * 2.0 ** -53 * 2.0 ** (2 * lg) * tot
    say(f"case lane anchor beyond n={n} k={split_k} lg={lg}: rel={abs(r.value - want) / want:.2e} tol={tol / want:.2e}")
    assert r.status == 0 and tol <= 1e-2 * want and abs(r.value - want) <= tol
    assert abs(r.sum_abs - tot) <= 8 * n * 2.0 ** -53 * 2.0 ** (2 * lg) * tot
