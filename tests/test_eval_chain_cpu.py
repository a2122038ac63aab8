"""The host's side of a lone evaluation's one chain, on the CPU (no GPU):
tests/schedsim/chain.cpp drives the host runtime, built against the HIP
stand-in, through recoveries from a failed root, also where the root slots
arrive after the result was announced, and through limits on device memory,
under AddressSanitizer with UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

from test_serving_scheduler_cpu import ROOT, SIM

SOURCES = [os.path.join(ROOT, "paper_2109_04528_amd", "csrc", "tor_runtime.cpp"),
           os.path.join(SIM, "fakehip.cpp"), os.path.join(SIM, "stubs.cpp"), os.path.join(SIM, "chain.cpp")]


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_chain_under_asan_and_ubsan(tmp_path):
    exe = str(tmp_path / "chain")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
                    "-I", os.path.join(SIM, "fake"), "-I", os.path.join(ROOT, "include"), *SOURCES, "-lpthread", "-Wl,--wrap=_Z9hipMallocPPvm",
                    "-o", exe],
                   check=True, capture_output=True, text=True, timeout=300)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1", UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stdout[-2000:], res.stderr[-4000:])
    assert res.stdout.strip().splitlines()[-1] == "done 0"
