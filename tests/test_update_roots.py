"""The square root and the reciprocal in the coefficients of the per-mode update
are the correctly rounded ones (host build of update.hpp)."""

import os
import subprocess

from paper_1608_05739_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


def test_roots_of_the_update_are_correctly_rounded(tmp_path):
    exe = str(tmp_path / "roots")
    # (4e6 arguments; one in 2^38 may differ)
    r = subprocess.run([B.hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-I", B.CSRC,
                        "-I", os.path.join(B.ROOT, "include"),
                        os.path.join(HERE, "host_update", "roots_driver.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout
