"""Plans that replay a captured step graph compute exactly what enqueued kernels
compute: batches whose passes have several launches, in 2D and 3D, with eager
work and synchronizations between the replays, each replay checked."""

import pytest

import fixtures
import oracle
import paper_1608_05739_amd as pk
from gpu_support import (GROUP_TOL, compare, fields_to_device, from_device, np_dtype, rounded, say,
                         to_device)

pytestmark = pytest.mark.gpu

SHAPES = {2: [(96, 64), (64, 128), (54, 96), (128, 48), (64, 64)],
          3: [(32, 48, 64), (64, 32, 48), (36, 64, 96), (48, 54, 32)]}  # (z[, y], x)


def _batch(ndim):
    parts = [fixtures.workload(ndim - 1, shape=s, steps=4) for s in SHAPES[ndim]]
    w = parts[0]
    for o in parts[1:]:
        w.patches, w.E0, w.B0 = w.patches + o.patches, w.E0 + o.E0, w.B0 + o.B0
        w.schedule = w.schedule + o.schedule
    return w


def _sources(plan, w, n, precision):
    srcs = [s.sources(n, dtype=np_dtype(precision)) for s in w.schedule]
    J = [to_device([s[0][c] for s in srcs], plan, precision) for c in range(3)]
    return J, to_device([s[1] for s in srcs], plan, precision), to_device([s[2] for s in srcs], plan, precision)


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("profiled", [False, True])
def test_every_replay_equals_enqueued_kernels(ndim, precision, profiled):
    import torch
    w = _batch(ndim)
    eager = pk.Plan(w.patches, precision=precision, source_mode="rho")
    graph = pk.Plan(w.patches, precision=precision, source_mode="rho", graph=True)
    assert "step=kernels" in eager.info.splitlines()[0] and "step=graph" in graph.info.splitlines()[0]
    say(f"graph {ndim}D {precision} profiled={profiled}")
    a = fields_to_device(w.E0, eager, precision) + fields_to_device(w.B0, eager, precision)
    b = [t.clone() for t in a]
    for n in range(4):
        J, ro, rn = _sources(eager, w, n, precision)
        eager.push(a[:3], a[3:], J, ro, rn)
        torch.cuda.synchronize()
        # the graph serves whatever buffers a push names: fresh ones every second step
        if n % 2:
            b = [t.clone() for t in b]
        push = graph.push_profiled if profiled else graph.push
        push(b[:3], b[3:], [j.clone() for j in J], ro.clone(), rn.clone())
        torch.cuda.synchronize()
        for x, y in zip(a, b):
            assert torch.equal(x, y), (n, ndim, precision)
    eager.close()
    graph.close()


def test_one_launch_per_pass_is_enqueued():
    p = pk.Patch(2, (64, 1, 96), (1.0, 1.0, 1.0), 0.5)
    plan = pk.Plan([p], graph=True)
    assert "step=kernels" in plan.info.splitlines()[0]
    plan.close()


@pytest.mark.parametrize("cdt", [5.0, 20.0])
@pytest.mark.parametrize("precision,path", [("fp32", "fused"), ("fp64", "plain")])
def test_3d_large_time_step_on_the_generic_kernels(cdt, precision, path):
    """c dt = 5 dx and 20 dx with sources on the generic 3D kernels, 3 steps."""
    w = fixtures.workload(2, shape=(48, 32, 64), steps=3)
    p0, s = w.patches[0], w.schedule[0]
    p = fixtures.workloads.Patch(3, p0.nx, p0.ny, p0.nz, p0.dx, p0.dy, p0.dz, cdt * p0.dx)
    sched = fixtures.SourceSchedule(s.P, s.D, s.phases, p.dt)
    plan = pk.Plan([p], precision=precision, source_mode="rho", path=path, generic_kernels=True)
    assert all("kernel=generic" in ln for ln in plan.info.splitlines()[1:] if ln.strip())
    say(f"generic 3D c dt = {cdt} dx {precision} {path}")
    E, B = fields_to_device(w.E0, plan, precision), fields_to_device(w.B0, plan, precision)
    w.schedule = [sched]
    for n in range(3):
        plan.push(E, B, *_sources(plan, w, n, precision))
    got = ([[from_device(t, plan)[0] for t in E]], [[from_device(t, plan)[0] for t in B]])
    plan.close()
    Eo, Bo = oracle.psatd_run([rounded(a, precision) for a in w.E0[0]],
                              [rounded(a, precision) for a in w.B0[0]], 3, d=p.d, dt=p.dt,
                              schedule=sched, source_dtype=np_dtype(precision))
    err = compare(got, ([Eo], [Bo]), precision=precision)
    assert err < GROUP_TOL[precision]
