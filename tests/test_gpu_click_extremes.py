"""Click probabilities at the ends of the range (GPU): states of which one
mode's block of I - O is so large that its determinant is no double, for the
patterns without that mode (the others' terms are no doubles either), against
the closed form of a product state; and a diagonal entry of -inf, which is an
invalid value only for the patterns that hold its mode."""
import sys

import numpy as np
import pytest

from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# O = diag(o, o): p(S) = prod over S of o_i, over the others of 1 - o_i, at a few roundings a mode
@pytest.mark.parametrize("M", [1, 3, 9, 12, 15])
@pytest.mark.parametrize("big", [1e100, 1e160, 1e200, 1e300])
@pytest.mark.parametrize("at", [0, -1])
def test_large_pivot(M, big, at):
    from paper_2109_04528_amd import Context
    o = np.full(M, 0.5)
    o[at] = -big
    want = np.ones(1)
    for x in o:
        want = np.concatenate([want * (1.0 - x), want * x])
    O = np.diag(np.concatenate([o, o])).astype(complex)
    say(f"case large pivot M={M} {big} at {at}")
    with Context() as ctx:
        p, _, _ = ctx.click_all(O)
        without = np.flatnonzero(((np.arange(1 << M) >> (at % M)) & 1) == 0)
        # the subset sums cancel to 2^(M-1) of their terms at most
        assert np.all(np.abs(p - want)[without] <= 64 * M * 2.0 ** (M - 53) * np.abs(want)[without])
        S = [0, int(without[-1]), int(without[len(without) // 2])]
        q, rs = ctx.click_probs(O, S)
        assert np.all(np.abs(q - want[S]) <= 64 * M * 2.0 ** (M - 53) * np.abs(want[S]))


@pytest.mark.parametrize("M", [1, 3, 9, 12, 26])
@pytest.mark.parametrize("mode", [0, -1])
@pytest.mark.parametrize("half", [0, 1])
def test_infinite_diagonal_entry(M, mode, half):
    from paper_2109_04528_amd import Context, TOR_E_INVAL, TorError
    O = gen.random_O(M, M, 0.8, 1.2, 0.8)
    m = mode % M
    O[m + half * M, m + half * M] = -np.inf
    say(f"case infinite diagonal entry M={M} mode={m} half={half}")
    with Context() as ctx:
        with pytest.raises(TorError) as ei:
            ctx.click_all(O)
        assert ei.value.code == TOR_E_INVAL
        others = [q for q in range(M) if q != m][:5]
        S = [0, 1 << m, sum(1 << q for q in others)]
        p, rs = ctx.click_probs(O, S, check=False)
        assert rs[0].status == 0 and rs[0].value == 1.0 and p[0] == np.inf
        assert rs[1].status == TOR_E_INVAL and np.isnan(p[1])
        if others:
            want = ctx.eval(gen.click_submatrix(O, others))
            assert rs[2].status == 0 and (rs[2].tor, rs[2].tor_lo) == (want.tor, want.tor_lo) and p[2] == np.inf
