"""A lone evaluation of up to 64 roots is summed by the wave that ends last,
more by the reduction kernel: both give the record of a batch of one at the
same split, bit for bit, also where the sum is not exact, on either path, with
the library's own workspace (the result is announced before the other path's
kernel has looked at the verdict) and a caller's (after it)."""
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


# 2, 32, 64, 128 roots
@pytest.mark.parametrize("k", [1, 5, 6, 7])
@pytest.mark.parametrize("accum", ["dd", "fp64"])
def test_sum_of_few_roots(k, accum):
    import torch
    from paper_2109_04528_amd import Context, TOR_INPUT_DEVICE
    n = 18  # seven levels above the leaves on the real path, nine on the complex one
    state, general = gen.random_O(n, 90 + k, 0.3, 1.2, 0.9), gen.random_hpd_O(n, 90 + k)
    # a real matrix whose subset determinants exceed 1: its sums are rounded
    rounded = state.copy()
    rounded[np.diag_indices(2 * n)] -= 2.0
    ws = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
    mats = [state, general, rounded, general, state, state]
    dev = [torch.from_numpy(O).cuda() for O in mats]
    torch.cuda.synchronize()
    with Context(split_k=k, accum=accum) as ref:
        want = [bits(ref.eval_batch([O])[0]) for O in mats]
        assert [w[5] for w in want] == [1, 2, 1, 2, 1, 1]
        say(f"case few roots k={k} {accum} host")
        assert [bits(ref.eval(O)) for O in mats] == want
    for kw in ({}, {"workspace": ws}):
        say(f"case few roots k={k} {accum} device {list(kw)}")
        with Context(split_k=k, accum=accum, flags=TOR_INPUT_DEVICE, **kw) as ctx:
            for _ in range(3):
                assert [bits(ctx.eval(O)) for O in dev] == want
