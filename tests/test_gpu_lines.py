"""The line passes with compile-time lengths against the oracle: every compiled
length as x rows (nx = 2 L), as y lines and as plain z lines, in both storage
precisions, with line counts that leave a short last tile.

Tolerances are the parity ones: one step differs from the oracle by FP64
rounding (about 1e-15 sqrt(log L), bound 1e-12) or by FP32 storage (a few
2^-24, bound 1e-5)."""

import pytest

import fixtures
import paper_1608_05739_amd as pk
from gpu_support import compare, run_gpu, run_oracle, say

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5}
LENGTHS = [24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 256, 288, 324, 384, 432,
           486, 512, 576, 648, 768, 864, 1024, 1152, 1296, 1536, 1728, 2048]


def _check(index, shape, precision, names, path):
    w = fixtures.workload(index, shape=shape, steps=2)
    plan = pk.Plan(w.patches, precision=precision, source_mode="rho", path=path)
    lines = {ln.split()[0]: ln for ln in plan.info.splitlines()[1:]}
    plan.close()
    want = "kernel=wave" if precision == "fp32" else "kernel=compile-time"
    assert all(lines[n].endswith(want) for n in names), lines
    say(f"fixed lines {shape} {precision}")
    err = compare(run_gpu(w, precision, path, w.steps), run_oracle(w, precision, w.steps),
                  precision=precision)
    assert err < TOL[precision]


@pytest.mark.parametrize("L", LENGTHS)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_every_line_length(L, precision):
    # 18 rows: a full tile of 16 or 8 and a short one
    _check(1, (18, 2 * L), precision, ["x_r2c_fwd", "x_c2r_inv"], "plain")
    _check(1, (L, 54), precision, ["z_c2c_fwd", "z_c2c_inv"], "plain")
    if L <= 1024:
        _check(2, (18, L, 6), precision, ["y_c2c_fwd", "y_c2c_inv"], "plain")


def test_choices_saved_with_earlier_tiles_still_apply():
    # tuning strings saved when the line kernels had other tiles
    p = pk.Patch(2, (64, 1, 96), (1.0, 1.0, 1.0), 0.5)
    for precision, text in (
            ("fp32", "psatd-tuning-1;7,0,64,0,0,-1;6,0,8,0,0,-1;7,0,64,0,0,4"),
            ("fp64", "psatd-tuning-1;0,1,96,0,0,0;1,0,8,2,0,-1;0,1,96,0,0,-1")):
        now = pk.Plan([p], precision=precision)
        again = pk.Plan([p], precision=precision, tuning=text)
        kinds = [[ln.split("kernel=")[1].split()[0] for ln in q.info.splitlines()[1:]]
                 for q in (now, again)]
        now.close()
        again.close()
        assert kinds[0][0] == kinds[1][0] and kinds[0][2] == kinds[1][2], kinds
