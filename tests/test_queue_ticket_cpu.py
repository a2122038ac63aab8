"""The queue of subtree roots hands every root out once whatever the compiler
does with atomics of many lanes (no GPU): with its merging of them switched
off, each atomic addition of a recursive kernel still runs under the mask of
one lane, right below the branch that sets it."""
import os
import subprocess

import pytest

from paper_2109_04528_amd import build

SINGLE = "s_and_saveexec_b64"


@pytest.mark.parametrize("source", ["tor_kernels.hip", "tor_kernels_quad.hip"])
def test_queue_atomics_of_one_lane(tmp_path, source):
    asm = tmp_path / "k.s"
    cmd = [build.hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-fno-fast-math", "-I", os.path.join(build.HERE, "..", "include"), "-mllvm",
           "-amdgpu-atomic-optimizer-strategy=None", "--cuda-device-only", "-S", "-x", "hip",
           os.path.join(build.CSRC, source), "-o", str(asm)]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    lines = asm.read_text().splitlines()
    found, kernel = 0, ""
    for i, line in enumerate(lines):
        if line.startswith("_Z") and line.split(";")[0].rstrip().endswith(":"):
            kernel = line
        if "tor_main" not in kernel or "global_atomic_add_x2" not in line:
            continue
        found += 1
        # back to where the execution mask was last changed or joined
        above = next(x for x in reversed(lines[:i]) if SINGLE in x or x.startswith(".LBB") or "_b64 exec, exec" in x)
        assert SINGLE in above, (kernel, i, above)
    assert found >= 3  # two of the queue and one of the finished roots, in every kernel
