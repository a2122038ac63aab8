"""A caller's workspace that holds the launch of the path a matrix takes, but
not room for either path's at once (GPU): the evaluation goes through the
general path and gives the same record; below what that path needs it is
TOR_E_NOMEM and the record stays untouched.  Sizes as the library lays its
workspace out."""
import sys

import pytest

from paper_2109_04528_amd import inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def nsz(s):
    return 2 * s * (s + 1)


def up(v):
    return (v + 255) // 256 * 256


def stack_bytes(N, k, R, scalar, real):
    gsum = lambda s: 0 if s <= 0 else 2 * s * (s + 1) * (s + 2) // 3
    LA = N - R
    slots = nsz(N) + gsum(N - k - 1) - gsum(N - LA) if k < LA else nsz(N)
    return up(scalar * slots + real * (LA + 1))


def launch(N, k, R, scalar, real, waves):
    """Root slots, descriptors (twice), the counter and the whole grid's stacks."""
    return up(32 << k) + 256 * 3 + stack_bytes(N, k, R, scalar, real) * waves


# real path: depths of 2048 waves; the complex path's room is what does not fit
@pytest.mark.parametrize("n,k", [(20, 9), (22, 11), (24, 11)])
@pytest.mark.parametrize("where", ["host", "device"])
def test_one_path_fits(where, n, k):
    import torch
    from paper_2109_04528_amd import Context, TOR_INPUT_DEVICE
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus != 256:
        pytest.skip("the depths are those of 256 CUs")
    flags = TOR_INPUT_DEVICE if where == "device" else 0
    O = gen.random_O(n, n, 0.3, 1.2, 0.9)
    x = torch.from_numpy(O).cuda() if flags else O
    # the staged form is sized for either path; a host matrix is read in place,
    # descriptors in pinned memory
    form = up(16 * nsz(n))
    real = form + launch(n, k, 11, 8, 8, 8 * cus)
    both = form + launch(n, min(n - 9, 11), 9, 16, 8, 8 * cus)
    assert real + 4096 < both  # so the room below is too small for the one chain
    with Context(flags=flags) as ref:
        want = ref.eval(x)
    for room, fits in ((real, True), (real + 4096, True), (real - 4096, False), (real // 2, False)):
        say(f"case small memory {where} n={n} room={room} fits={fits}")
        ws = torch.empty(room, dtype=torch.uint8, device="cuda")
        with Context(flags=flags, workspace=ws) as ctx:
            if fits:
                r = ctx.eval(x)
                assert (r.tor, r.tor_lo, r.sum_abs, r.status, r.path) == (want.tor, want.tor_lo, want.sum_abs, 0, 1)
                assert r.device_ms > 0.0
            else:
                from paper_2109_04528_amd import TOR_E_NOMEM, TorError
                with pytest.raises(TorError) as ei:
                    ctx.eval(x)
                assert ei.value.code == TOR_E_NOMEM
