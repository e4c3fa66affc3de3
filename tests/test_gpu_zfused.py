"""The fused z pass with compile-time lengths against the oracle: every compiled
length in 2D (all forms, both precisions, PSTD) and 3D, with line counts that
leave a short last item.

Tolerances are the parity ones (see test_gpu_lines.py): FP64 1e-12, FP32 1e-5."""

import numpy as np
import pytest

import fixtures
import oracle.contrast
import paper_1608_05739_amd as pk
from gpu_support import compare, fields_to_device, from_device, run_gpu, run_oracle, say, to_device

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5}
LENGTHS_3D = [32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 256, 288, 324, 384, 432, 512]
LENGTHS_2D = LENGTHS_3D + [576, 648, 768, 864, 1024, 1152, 1296, 1536, 1728, 2048, 2304, 3072, 4096]


def _check(index, shape, precision, form):
    if form == "vacuum":
        w = fixtures.workload(index, shape=shape, steps=2)
        w.sources = False
    else:
        w = fixtures.workload(index, shape=shape, steps=2)
    mode = {"rho": "rho", "J": "j", "vacuum": "vacuum"}[form]
    plan = pk.Plan(w.patches, precision=precision, source_mode=mode, path="fused")
    info = plan.info
    plan.close()
    line = [ln for ln in info.splitlines() if ln.strip().startswith("z_fused")][0]
    assert line.endswith("kernel=wave" if precision == "fp32" else "kernel=compile-time"), info
    say(f"fixed z {shape} {precision} {form}")
    f = form if form != "vacuum" else "rho"
    err = compare(run_gpu(w, precision, "fused", w.steps, form=f), run_oracle(w, precision, w.steps, form=f),
                  precision=precision)
    assert err < TOL[precision]


@pytest.mark.parametrize("L", LENGTHS_2D)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_2d_every_z_length_and_form(L, precision):
    if precision == "fp64" and L > 2048:
        pytest.skip("FP64 plans run the plain z passes above 2048 points")
    for form in ("rho", "J", "vacuum"):
        _check(1, (L, 54), precision, form)  # 27 columns


@pytest.mark.parametrize("L", LENGTHS_3D)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_3d_every_z_length_and_form(L, precision):
    for form in ("rho", "J", "vacuum"):
        if precision == "fp64" and form == "rho" and L % 3 == 0 and L not in (54, 162, 324):
            continue  # generic kernel
        _check(2, (L, 6, 6), precision, form)  # 18 lines


@pytest.mark.parametrize("L", [64, 96, 162, 1024, 2304])
@pytest.mark.parametrize("mode", ["vacuum", "j"])
def test_pstd_sets(L, mode):
    import torch
    w = fixtures.workload(1, shape=(L, 48), steps=2)
    p = w.patches[0]
    p.dt *= 0.4
    plan = pk.Plan([p], precision="fp32", source_mode=mode, pstd=True)
    assert "kernel=wave" in [ln for ln in plan.info.splitlines() if "z_fused" in ln][0]
    E, B = fields_to_device(w.E0, plan, "fp32"), fields_to_device(w.B0, plan, "fp32")
    r32 = lambda v: [np.asarray(a, np.float32).astype(np.float64) for a in v]  # noqa: E731
    J = r32(w.schedule[0].sources(0)[0]) if mode == "j" else None
    Eo, Bo = oracle.contrast.pstd_step(r32(w.E0[0]), r32(w.B0[0]), J, d=p.d, dt=p.dt)
    plan.push(E, B, [to_device([j], plan, "fp32") for j in J] if J else None)
    torch.cuda.synchronize()
    got = [from_device(t, plan)[0] for t in E + B]
    plan.close()
    ref = list(Eo) + list(Bo)
    err = np.sqrt(sum(np.sum((g - r) ** 2) for g, r in zip(got, ref)) / sum(np.sum(r * r) for r in ref))
    say(f"pstd sets {L} {mode}: {err:.1e}")
    assert err < TOL["fp32"]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("mode", ["vacuum", "rho", "j"])
@pytest.mark.parametrize("graph", [False, True])
def test_families_of_lengths_equal_patches_alone(precision, mode, graph):
    """A batch with several 2^k and 3 2^k z lengths runs each family in one launch;
    a patch alone runs the kernel of its length.  27, 6 and 36 columns leave a short
    last item at every length.  Both round the same FP64 arithmetic to storage at the
    same places, so they differ by its last bits at most: the bounds are a few
    rounding units of the storage."""
    import torch
    lengths = [32, 512, 48, 72, 64, 384, 54, 128, 192, 256, 96, 144]
    patches = [pk.Patch(2, ((54, 12, 72)[i % 3], 1, L), (1 / 32,) * 3, 1 / 40) for i, L in enumerate(lengths)]
    dtype = torch.float32 if precision == "fp32" else torch.float64
    gen = torch.Generator().manual_seed(7)
    ncomp = {"vacuum": 6, "j": 9, "rho": 11}[mode]
    batch = pk.Plan(patches, precision=precision, source_mode=mode, graph=graph)
    data = torch.randn(ncomp, batch.total_elements, generator=gen, dtype=torch.float64).to(dtype)

    def push(plan, comps):
        t = [c.clone().cuda() for c in comps]
        args = [t[0:3], t[3:6]] + ([t[6:9]] if ncomp > 6 else []) + (t[9:11] if ncomp > 9 else [])
        plan.push(*args)
        torch.cuda.synchronize()
        return [x.cpu().double() for x in t[:6]]

    say(f"z families {precision} {mode} graph={graph}")
    got = push(batch, data)
    offsets = batch.offsets
    batch.close()
    bound = 5e-7 if precision == "fp32" else 1e-14
    for p, off in zip(patches, offsets):
        alone = pk.Plan([p], precision=precision, source_mode=mode)
        n = alone.total_elements
        ref = push(alone, data[:, off:off + n])
        alone.close()
        for a, b in zip(got, ref):
            d = torch.linalg.vector_norm(a[off:off + p.cells] - b[:p.cells])
            assert d <= bound * torch.linalg.vector_norm(b[:p.cells]), (p, float(d))


@pytest.mark.parametrize("shape", [(1024, 8), (2048, 8), (4096, 4), (1536, 6), (3072, 2)])
@pytest.mark.parametrize("form", ["rho", "J"])
def test_long_lines_of_few_columns_in_a_batch(shape, form):
    """1 to 4 columns leave most of a work item of long lines idle."""
    w, other = fixtures.workload(1, shape=shape, steps=2), fixtures.workload(1, shape=(96, 54), steps=2)
    w.patches, w.E0, w.B0 = w.patches + other.patches, w.E0 + other.E0, w.B0 + other.B0
    w.schedule = w.schedule + other.schedule
    plan = pk.Plan(w.patches, source_mode={"rho": "rho", "J": "j"}[form])
    assert [ln for ln in plan.info.splitlines() if "z_fused" in ln][0].endswith("kernel=wave"), plan.info
    plan.close()
    say(f"few columns {shape} {form}")
    err = compare(run_gpu(w, "fp32", "fused", 2, form=form), run_oracle(w, "fp32", 2, form=form))
    assert err < TOL["fp32"]


def test_3d_saved_choice_of_the_other_z_kernel():
    """96 x 64 x 64 runs the generic z kernel by default; a saved choice of the
    compile-time one (32 lines per work item) applies, and agrees with it."""
    import torch
    p = pk.Patch(3, (64, 64, 96), (1 / 32,) * 3, 1 / 40)
    plain = pk.Plan([p], source_mode="rho")
    choices = plain.tuning.split(";")
    assert choices[3].split(",")[0] == "1"
    choices[3] = "6,0,32,0,0,-1"
    other = pk.Plan([p], source_mode="rho", tuning=";".join(choices))
    say("3D saved z choice")
    out = []
    for plan in (plain, other):
        g = torch.Generator().manual_seed(3)
        t = [torch.randn(plan.total_elements, generator=g).cuda() for _ in range(11)]
        plan.push(t[0:3], t[3:6], t[6:9], t[9], t[10])
        torch.cuda.synchronize()
        out.append(torch.cat([x.double() for x in t[:6]]))
        plan.close()
    # the same FP64 arithmetic rounded to FP32 storage at the same places
    assert torch.linalg.vector_norm(out[0] - out[1]) <= 5e-7 * torch.linalg.vector_norm(out[0])
