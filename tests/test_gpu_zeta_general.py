"""The subset-sum transform beyond the domain in which every sum is exact
(GPU): terms of any size and sign, and states so bright that partial sums pass
2^53.  Each addition keeps both low parts: the sums have the bits of the same
additions made of Knuth's TwoSum alone, in the kernels' order, and their errors
stay within 3 * 2^-106 of each partial sum."""
import sys
from fractions import Fraction

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


def two_sum(a, b):
    s = a + b
    bb = s - a
    return s, (a - (s - bb)) + (b - bb)


def add(ah, al, bh, bl):
    s, e = two_sum(ah, bh)
    t, f = two_sum(al, bl)
    s, e = two_sum(s, e + t)
    return two_sum(s, e + f)


def first_stage(nb):
    """Index bits in the order a workgroup adds along them: groups of registers
    from the highest down, or one by one."""
    group = {12: 4, 10: 2}.get(nb)
    return [s + b for s in range(nb - group, -1, -group) for b in range(group)] if group else list(range(nb))


def tile(b0, w):
    cb = 12 - w
    return [b0 + i - cb for i in [8, 9, 10, 11] + ([4, 5, 6, 7] if cb < 8 else []) if i >= cb]


def middle(b0, b1):
    order = []
    while b0 < b1:
        left = b1 - b0
        w = left if left <= 8 else left - 8 if left <= 13 else 8
        order += list(range(b0, b0 + w)) if w <= 5 else tile(b0, w)
        b0 += w
    return order


def transform(t, order):
    h, l = t.copy(), np.zeros_like(t)
    for b in order:
        h, l = h.reshape(-1, 2, 1 << b), l.reshape(-1, 2, 1 << b)
        h[:, 1], l[:, 1] = add(h[:, 1], l[:, 1], h[:, 0], l[:, 0])
        h, l = h.reshape(-1), l.reshape(-1)
    return h, l


def terms(n, seed):
    rng = np.random.default_rng(seed)
    return rng.choice([-1.0, 1.0], n) * rng.uniform(1.0, 2.0, n) * 2.0 ** rng.integers(0, 60, n)


# one bit at a time (9, 11), in registers (10, 12), register passes (13, 17), tiles (18, 20), both (21)
@pytest.mark.parametrize("nbits", [9, 10, 11, 12, 13, 17, 18, 20, 21])
def test_bits_of_the_general_addition(ctx, nbits):
    t = terms(1 << nbits, nbits)
    nb = min(nbits, 12)
    h, l = transform(t, first_stage(nb) + middle(nb, nbits))
    hi, lo = ctx.debug_zeta(t)
    say(f"case general transform nbits={nbits}")
    assert np.array_equal(hi, h) and np.array_equal(lo, l)


def test_error_of_every_sum(ctx):
    t = terms(1 << 10, 5)
    hi, lo = ctx.debug_zeta(t)
    exact, err = [Fraction(float(x)) for x in t], [Fraction(0)] * (1 << 10)
    for b in first_stage(10):
        for i in range(1 << 10):
            if (i >> b) & 1:
                exact[i] += exact[i ^ (1 << b)]
                err[i] += err[i ^ (1 << b)]
                # 3u^2 of the computed sum, itself within err of the exact one
                err[i] += Fraction(4, 1 << 106) * (abs(exact[i]) + err[i])
    say("case general transform error")
    for i in range(1 << 10):
        assert abs(Fraction(float(hi[i])) + Fraction(float(lo[i])) - exact[i]) <= err[i]


# the pattern pass takes 0, 4, 7 and 8 of the bits
@pytest.mark.parametrize("M", [12, 14, 17, 20])
def test_bright_states(ctx, M):
    O = gen.product_state_O(np.linspace(3.4, 4.4, M), 1.0)
    _, (th, tl), r = ctx.click_all(O, tor=True)
    assert r.sum_abs > 2.0 ** 55  # beyond the exact sums' domain
    # the sums by index (pattern S's is at its bits reversed) without their signs
    S = np.arange(1 << M)
    rev = sum(((S >> q) & 1) << (M - 1 - q) for q in range(M))
    sign = np.where((M - sum((S >> q) & 1 for q in range(M))) % 2, -1.0, 1.0)
    gh, gl = np.empty(1 << M), np.empty(1 << M)
    gh[rev], gl[rev] = sign * th, sign * tl
    # the terms: differences along every bit, to far less than a term's last bit
    h, l = gh.copy(), gl.copy()
    for b in range(M):
        h, l = h.reshape(-1, 2, 1 << b), l.reshape(-1, 2, 1 << b)
        h[:, 1], l[:, 1] = add(h[:, 1], l[:, 1], -h[:, 0], -l[:, 0])
        h, l = h.reshape(-1), l.reshape(-1)
    last = min(M - 10, 8)
    order = first_stage(12) if M == 12 else first_stage(10 if M - last <= 10 else 12) + tile(M - last, last)
    eh, el = transform(h, order)
    say(f"case bright state M={M} sum_abs=2^{np.log2(r.sum_abs):.1f}")
    assert np.array_equal(eh, gh) and np.array_equal(el, gl)
