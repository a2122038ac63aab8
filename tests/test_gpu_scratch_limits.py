"""Where the scratch is given and small, a launch takes fewer waves and smaller
per-wave stacks: the static array holds every path up to 30 modes (31 on the
16-byte paths, not 32), and a caller's workspace that holds 7 waves per CU at
the deeper split still serves, alone and in a batch."""
import sys

import pytest

from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("flag,n", [("TOR_FORCE_COMPLEX", 30), ("TOR_FORCE_COMPLEX", 31), ("TOR_FACTOR_DD", 29),
                                    ("TOR_FACTOR_DD", 30), ("TOR_FACTOR_DD", 31)])
def test_static_array_holds_the_16_byte_paths(flag, n):
    import paper_2109_04528_amd as tor
    O = gen.random_O(n, 30 + n, 0.5, 1.0, 0.7)
    say(f"case static scratch {flag} n={n}")
    with tor.Context(flags=getattr(tor, flag)) as ctx:
        r, want = ctx.eval_static(O), ctx.eval(O)
        assert r.status == 0
        # a Gaussian state's FP64 terms sum exactly, whatever the split; the
        # double-double ones to 2^-90 of the sum of their magnitudes
        if flag == "TOR_FACTOR_DD":
            assert abs((r.tor - want.tor) + (r.tor_lo - want.tor_lo)) <= 2.0 ** -90 * want.sum_abs
        else:
            assert (r.tor, r.tor_lo) == (want.tor, want.tor_lo)
        with pytest.raises(tor.TorError) as ei:
            ctx.eval_static(gen.random_O(32, 1, 0.5, 1.0, 0.7))
        assert ei.value.code == tor.TOR_E_SCRATCH


def nsz(s):
    return 2 * s * (s + 1)


def stack_bytes(N, k, R, scalar, real):
    gsum = lambda s: 0 if s <= 0 else 2 * s * (s + 1) * (s + 2) // 3
    LA = N - R
    slots = nsz(N) + gsum(N - k - 1) - gsum(N - LA) if k < LA else nsz(N)
    return (scalar * slots + real * (LA + 1) + 255) // 256 * 256


# the depths of about 32 leaves per root, from one root for every second wave on
@pytest.mark.parametrize("flag,real", [("TOR_FORCE_COMPLEX", 8), ("TOR_FACTOR_DD", 16)])
@pytest.mark.parametrize("n", [18, 22, 26])
def test_small_workspace_with_seven_waves(flag, real, n):
    import torch
    import paper_2109_04528_amd as tor
    fl = getattr(tor, flag) | tor.TOR_INPUT_DEVICE
    O = torch.from_numpy(gen.random_O(n, 30 + n, 0.5, 1.0, 0.7)).cuda()
    LA = n - 9
    k = min(LA, max(10, min(14, LA - 5)))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    room = 4096 + 16 * nsz(n) + (32 << k) + 7 * cus * stack_bytes(n, k, 9, 16, real)
    say(f"case small workspace {flag} n={n} {room / 2 ** 20:.1f} MiB")
    ws = torch.empty(room, dtype=torch.uint8, device="cuda")
    with tor.Context(flags=fl) as ref, tor.Context(flags=fl, workspace=ws) as ctx:
        want, r = ref.eval(O), ctx.eval(O)
        assert r.status == 0
        assert abs((r.tor - want.tor) + (r.tor_lo - want.tor_lo)) <= 2.0 ** -90 * want.sum_abs
