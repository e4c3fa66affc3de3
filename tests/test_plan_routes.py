"""Which fused z kernel a plan runs by default (host-only planning): 3D lines at
12 points per thread run the generic kernel while it is done in one round of
workgroups, large batches of narrow patches run it, and one patch of few columns
does not decide for a batch."""

import pytest

import paper_1608_05739_amd as pk


def z_kernel(shapes, **kw):
    patches = [pk.Patch(3 if s[1] > 1 else 2, s, (1.0, 1.0, 1.0), 0.5) for s in shapes]
    info = pk.describe_plan(patches, **kw)[1]
    line = [ln for ln in info.splitlines() if ln.strip().startswith("z_fused")][0]
    return "generic" if line.endswith("kernel=generic") else "fixed"


@pytest.mark.parametrize("shape,precision,mode,want", [
    ((64, 64, 96), "fp32", "rho", "generic"),     # 2048 lines: 205 workgroups
    ((96, 64, 96), "fp32", "rho", "fixed"),       # 3072 lines: 308
    ((48, 32, 216), "fp64", "vacuum", "generic"), ((128, 64, 216), "fp64", "vacuum", "fixed"),
    ((256, 256, 96), "fp64", "j", "generic"), ((192, 96, 288), "fp64", "j", "fixed"),
    ((64, 64, 64), "fp32", "rho", "fixed"), ((64, 64, 54), "fp32", "rho", "fixed"),
    ((6, 6, 96), "fp32", "rho", "fixed")])
def test_3d_lines_of_12_points_per_thread(shape, precision, mode, want):
    assert z_kernel([shape], precision=precision, source_mode=mode) == want


def test_few_columns_do_not_decide_for_a_batch():
    for few in ((8, 1, 1024), (4, 1, 4096), (6, 1, 1536)):
        assert z_kernel([few], source_mode="rho") == "generic"
        assert z_kernel([few, (64, 1, 64)], source_mode="rho") == "fixed"
        assert z_kernel([few, few], source_mode="rho") == "generic"


@pytest.mark.parametrize("nx,nz,patches,mode,want", [
    (16, 96, 256, "rho", "generic"), (16, 96, 255, "rho", "fixed"), (16, 96, 511, "vacuum", "fixed"),
    (16, 96, 512, "vacuum", "generic"), (18, 96, 512, "rho", "fixed"), (16, 64, 256, "rho", "fixed"),
    (16, 64, 512, "rho", "generic"), (64, 64, 512, "rho", "fixed")])
def test_large_batches_of_narrow_patches(nx, nz, patches, mode, want):
    # 32 lines per work item at 64 and 96 points: 8 columns fill a quarter of one
    assert z_kernel([(nx, 1, nz)] * patches, source_mode=mode) == want
