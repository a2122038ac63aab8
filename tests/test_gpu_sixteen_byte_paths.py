"""The 16-byte paths with eight waves per CU: two nodes of the last breadth-first
level lie behind the live blocks of two earlier ones.  The 64 lanes of one leaf
(9 modes) read every stored node, alone and after other leaves and roots."""
import sys

import pytest

import bounds
from oracle import oracle as orc
from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# padded, one leaf, two leaves, several; one root and many
@pytest.mark.parametrize("n", [4, 8, 9, 10, 11, 13])
@pytest.mark.parametrize("k", [0, 1, 3])
def test_every_stored_node(n, k):
    from paper_2109_04528_amd import Context, TOR_FACTOR_DD
    say(f"case 16-byte paths n={n} k={k}")
    O = gen.random_hpd_O(n, 60 + n)
    q = orc.tor(O, mode=orc.QUAD)
    with Context(split_k=k) as ctx:
        r = ctx.eval(O)
    assert r.path == 2
    assert abs((r.tor - q.hi) + (r.tor_lo - q.lo)) <= bounds.sum_bound(q.sum_sq, bounds.U64, bounds.UQ)
    O = gen.random_O(n, 60 + n, 0.3, 1.2, 0.9)
    q = orc.tor(O, mode=orc.QUAD)
    with Context(split_k=k, flags=TOR_FACTOR_DD) as ctx:
        r = ctx.eval(O)
    assert r.path == 3
    tol = bounds.sum_bound(q.sum_sq, bounds.UDD, bounds.UQ) + 4 * bounds.UDD * abs(q.value)
    assert abs((r.tor - q.hi) + (r.tor_lo - q.lo)) <= tol
