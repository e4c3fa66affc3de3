"""Error of the compile-time transforms of the FP64 passes, on the host: the
driver runs the kernels' own stages (tests/host_transforms) for every compiled
length against a DFT in long double."""

import os
import subprocess

from paper_1608_05739_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host_transforms", "transform_error_driver.cpp")


def test_fp64_transforms_stay_within_their_rounding_bound(tmp_path):
    exes = [str(tmp_path / f"driver{part}") for part in range(4)]
    builds = [subprocess.Popen([B.hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-O1",
                                f"-DPART={part}", "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC,
                                SRC, "-o", exe], stderr=subprocess.PIPE, text=True)
              for part, exe in enumerate(exes)]
    for p in builds:
        err = p.communicate(timeout=600)[1]
        assert p.returncode == 0, err[-4000:]
    cases = 0
    for exe in exes:
        r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, "\n".join(ln for ln in r.stdout.splitlines() if "FAIL" in ln)
        assert r.stdout.strip().endswith("0 failed")
        cases += r.stdout.count("inverse")
    assert cases >= 31 + 29  # every line length, every FP64 z length in each way it takes twiddles
