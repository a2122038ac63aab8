"""The passes of the subset-sum transform (GPU): every split of the index bits
into a first stage, register passes and tiles, against exact integer sums; and
the pass that writes the patterns, against the closed form of a product
state."""
import sys

import numpy as np
import pytest

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


# 12 bits alone; 1 and 5 more in registers; 6, 7 and 8 by a tile; 1 + 8
@pytest.mark.parametrize("nbits", [11, 12, 13, 17, 18, 19, 20, 21])
def test_transform_against_integer_sums(ctx, nbits):
    rng = np.random.default_rng(nbits)
    # every partial sum stays below 2^52
    t = rng.integers(-(1 << 30), 1 << 30, size=1 << nbits)
    hi, lo = ctx.debug_zeta(t.astype(np.float64))
    g = t.copy()
    for b in range(nbits):
        g = g.reshape(-1, 2, 1 << b)
        g[:, 1] += g[:, 0]
        g = g.reshape(-1)
    say(f"case transform nbits={nbits}")
    assert np.all(lo == 0.0) and np.array_equal(hi.astype(np.int64), g)


# the pattern pass takes 3, 4, ... 8 bits after a first stage of 10 (M = 13 to
# 18), then 8 after 11 or 12 and after register passes
@pytest.mark.parametrize("M", [13, 14, 15, 16, 17, 18, 19, 20, 21, 23])
def test_patterns_of_a_product_state(ctx, M):
    # p(S) = prod over S of (1 - p0), over the others of p0, p0 = sqrt(det) of the
    # mode's own block: distinct modes, so a misplaced pattern shows
    r = np.linspace(1.2, 1.8, M)
    O = gen.product_state_O(r, 0.9)
    p0 = np.array([np.sqrt(np.linalg.det(np.eye(2) - O[np.ix_([q, q + M], [q, q + M])]).real) for q in range(M)])
    want = np.ones(1)
    for q in range(M):
        want = np.concatenate([want * p0[q], want * (1.0 - p0[q])])  # bit q above the lower ones
    p, (hi, lo), r_ = ctx.click_all(O, tor=True)
    # Sec. 5's error of a sum of 2^n terms of independent roundings: R u times a
    # few tens of operations; R = prod (1 + p0) / (1 - p0) at most
    tol = 100 * 2.0 ** -53 * np.prod((1.0 + p0) / (1.0 - p0)) + 1e-13
    err = np.max(np.abs(p - want) / want)
    say(f"case product state M={M} err={err:.2e} tol={tol:.2e}")
    assert tol < 1e-4 and err <= tol
    root = np.prod(p0)
    assert np.max(np.abs((hi + lo) * root - want) / want) <= tol
    assert r_.tor == hi[-1] and r_.tor_lo == lo[-1]
