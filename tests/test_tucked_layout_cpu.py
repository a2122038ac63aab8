"""The LDS layout of the 16-byte paths (no GPU): a tree whose pivots would lie
over blocks that are still read, or whose tucked nodes find no room, does not
compile."""
import os
import subprocess

import pytest

from paper_2109_04528_amd import build


# R = 9, BL = 4 is the layout in use (21 + 15 = 36 = NB(8)); at R = 8 the pivots
# would start at block 25 of the 28 that level 2 reads, at R = 10 a tucked node
# would need 49 of 45 blocks
@pytest.mark.parametrize("R,message", [(9, None), (8, "pivots behind the blocks"), (10, "room behind the live blocks")])
def test_layouts(tmp_path, R, message):
    src = tmp_path / "layout.hip"
    src.write_text(f'#define TOR_KERNELS_TEMPLATES_ONLY\n#include "{build.CSRC}/tor_kernels.hip"\n'
                   f'namespace tor {{ static_assert(TuckedPivots<c64, {R}, 4, 2>::AT > 0, ""); }}\n')
    cmd = [build.hipcc(), "--offload-arch=gfx950", "-std=c++17", "-I", os.path.join(build.HERE, "..", "include"), "-I", build.CSRC,
           "--cuda-device-only", "-fsyntax-only", "-x", "hip", str(src)]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    if message is None:
        assert res.returncode == 0, res.stderr[-2000:]
    else:
        assert res.returncode != 0 and message in res.stderr, res.stderr[-2000:]
