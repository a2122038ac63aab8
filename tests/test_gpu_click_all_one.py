"""click_all enqueued in one go: staging and sqrt(det(I - O)) in one launch at
the sizes where the staged form and the number of transform passes change, and
a call after one that failed on the way."""
import sys

import numpy as np
import pytest

from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# padded below 11 modes; one transform stage up to 12; tiles from 13; 16 entries
# a thread in the first stage from 19
@pytest.mark.parametrize("M", [1, 2, 10, 11, 12, 13, 18, 19])
@pytest.mark.parametrize("check", [False, True])
def test_same_vacuum_and_no_residue_of_a_failed_call(M, check):
    from paper_2109_04528_amd import Context, TOR_CHECK_HERMITIAN, TOR_E_NOT_PD, TorError
    O = gen.random_O(M, 400 + M, 0.3, 1.2, 0.9)
    say(f"case click_all in one go M={M} check={check}")
    with Context(flags=TOR_CHECK_HERMITIAN if check else 0) as ctx:
        with pytest.raises(TorError) as ei:
            ctx.click_all(O + 2.0 * np.eye(2 * M), tor=True)
        assert ei.value.code == TOR_E_NOT_PD
        p, (th, tl), r = ctx.click_all(O, tor=True)
        # the pattern of no clicks is sqrt(det(I - O)) alone, formed by the same
        # steps as a call for one pattern forms it
        q, _ = ctx.click_probs(O, [0])
        assert p[0] == q[0] and (th[0], tl[0]) == (1.0, 0.0)
        e = ctx.eval(O)
        assert (th[-1], tl[-1], r.sum_abs) == (e.tor, e.tor_lo, e.sum_abs)
        assert r.device_ms > 0.0
