"""tor_eval_static splits as tor_eval does: the same record bit for bit on
every path, also where the terms' sum is rounded (general Hermitian matrices,
the double-double factor) and up to the largest sizes the array holds."""
import sys

import pytest

from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("form,n", [("hermitian", 13), ("hermitian", 21), ("hermitian", 29), ("hermitian", 30), ("hermitian", 31),
                                    ("dd", 10), ("dd", 22), ("dd", 29), ("dd", 30), ("dd", 31), ("state", 31)])
def test_static_has_the_bits_of_eval(form, n):
    from paper_2109_04528_amd import Context, TOR_FACTOR_DD
    O = gen.random_hpd_O(n, n) if form == "hermitian" else gen.random_O(n, n, 0.5, 1.0, 0.7)
    say(f"case static split {form} n={n}")
    with Context(flags=TOR_FACTOR_DD if form == "dd" else 0) as ctx:
        a, b = ctx.eval_static(O), ctx.eval(O)
        assert a.status == 0 and a.path == {"state": 1, "hermitian": 2, "dd": 3}[form]
        assert (a.tor, a.tor_lo, a.sum_abs, a.path) == (b.tor, b.tor_lo, b.sum_abs, b.path)
