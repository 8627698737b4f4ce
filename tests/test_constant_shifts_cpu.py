"""The host side of the kernel sources has no shift by a negative or too large
constant in any template that is instantiated (launch sizes are computed there
from tile shapes). Compiled for syntax only."""
import glob
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2304_14969_amd", "csrc")


@pytest.mark.parametrize("source", sorted(os.path.basename(p) for p in glob.glob(CSRC + "/*.hip")))
def test_no_shift_out_of_range(source):
    from paper_2304_14969_amd import build
    r = subprocess.run([build.hipcc(), "--offload-arch=gfx950", "-std=c++17", f"-I{build.INCLUDE}",
                        "--cuda-host-only", "-fsyntax-only", "-Werror=shift-count-negative",
                        "-Werror=shift-count-overflow", "-x", "hip", os.path.join(CSRC, source)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
