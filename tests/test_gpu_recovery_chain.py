"""Recovery from a failed root in a lone evaluation's one chain (GPU): one root
(staged and evaluated by one launch), a few (summed by the last wave) and more
(the reduction kernel), on each path, from host and device memory; a recovered
result equals the clean one bit for bit."""
import sys

import pytest

from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def bits(r):
    return (r.tor, r.tor_lo, r.sum_abs, r.err_est, r.status, r.path)


@pytest.mark.parametrize("form", ["state", "hermitian", "dd"])
@pytest.mark.parametrize("n,root", [(9, 0), (14, 3), (17, 20), (20, 300)])
def test_recovered_equals_clean(form, n, root):
    import torch
    from paper_2109_04528_amd import Context, TOR_E_NUMERIC, TOR_FACTOR_DD, TOR_INPUT_DEVICE
    O = gen.random_hpd_O(n, n) if form == "hermitian" else gen.random_O(n, n, 0.3, 1.2, 0.9)
    flags = TOR_FACTOR_DD if form == "dd" else 0
    for fl, x in ((flags, O), (flags | TOR_INPUT_DEVICE, torch.from_numpy(O).cuda())):
        say(f"case chain recovery {form} n={n} root={root} flags={fl}")
        with Context(flags=fl) as ctx:
            clean = ctx.eval(x)
            assert clean.launches == 1
            ctx.debug_fail_root(root, runs=1)
            r = ctx.eval(x)
            assert r.launches == 2 and bits(r) == bits(clean)
            ctx.debug_fail_root(root, runs=2)
            r = ctx.eval(x, check=False)
            assert r.launches == 2 and r.status == TOR_E_NUMERIC
            r = ctx.eval(x)
            assert r.launches == 1 and bits(r) == bits(clean)
