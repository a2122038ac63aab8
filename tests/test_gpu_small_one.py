"""The smallest evaluations, staged and evaluated by one launch (up to 11 modes
on the real path, 9 on the others), and the sizes next to them: the record of a
batch of one, bit for bit, also after inputs that are refused."""
import sys

import numpy as np
import pytest

from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def bits(r):
    return (r.tor, r.tor_lo, r.sum_abs, r.err_est, r.status, r.path, r.subsets, r.launches)


@pytest.mark.parametrize("n", [1, 2, 8, 9, 10, 11, 12])
@pytest.mark.parametrize("flag", [0, "TOR_CHECK_HERMITIAN", "TOR_FORCE_COMPLEX", "TOR_FACTOR_DD"])
def test_smallest_equal_batch_of_one(n, flag):
    import torch
    import paper_2109_04528_amd as tor
    fl = getattr(tor, flag) if flag else 0
    state = gen.random_O(n, 700 + n, 0.3, 1.2, 0.9)
    mats = [state] if flag == "TOR_FACTOR_DD" else [state, gen.random_hpd_O(n, 700 + n), state]
    bad = state.copy()
    bad[2 * n - 1, 0] = np.nan
    say(f"case smallest n={n} {flag}")
    with tor.Context(flags=fl) as h, tor.Context(flags=fl | tor.TOR_INPUT_DEVICE) as d:
        want = [bits(h.eval_batch([O])[0]) for O in mats]
        assert all(w[4] == 0 for w in want)
        for ctx, put in ((h, lambda O: O), (d, lambda O: torch.from_numpy(O).cuda())):
            with pytest.raises(tor.TorError) as ei:
                ctx.eval(put(bad))
            assert ei.value.code == tor.TOR_E_INVAL
            with pytest.raises(tor.TorError) as ei:
                ctx.eval(put(state + 2.0 * np.eye(2 * n)))
            assert ei.value.code == tor.TOR_E_NOT_PD
            assert [bits(ctx.eval(put(O))) for O in mats] == want
