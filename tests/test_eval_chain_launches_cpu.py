"""The launches of a lone evaluation's chain (no GPU): tests/chainsim links the
built library with a hipLaunchKernel of its own and checks, over the numbers of
roots on either path, that nothing is enqueued behind the launch that announces
the end, and that this launch announces it whatever the verdict."""
import os
import subprocess

import pytest

from paper_2109_04528_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_only_the_last_launch_announces(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path / "launches")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc())))
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=alignas(n)", "-I", os.path.join(rocm, "include"),
                    os.path.join(HERE, "chainsim", "launches.cpp"), "-Wl,--no-as-needed", build.LIB, "-L", os.path.join(rocm, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.dirname(build.LIB), "-Wl,-rpath," + os.path.join(rocm, "lib"), "-o", exe],
                   check=True, capture_output=True, text=True, timeout=120)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stderr[-3000:]
