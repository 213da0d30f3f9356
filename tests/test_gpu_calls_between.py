"""Other calls between the steps of a run leave the run as it was.

A run's pending force may lie in element-local forces while semx_step is under
way.  Force applies (direct, or replayed from a graph that the caller captured),
new sources, and switches of the assembly between two semx_step calls must
give the same state as stepping without graphs and without such applies.
"""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import rel_l2

pytestmark = pytest.mark.gpu

N = 5
CHUNK = 8
CALLS = 4          # semx_step calls of STEPS steps each
STEPS = 2 * CHUNK + 5


def _run(between, chunk):
    """State after CALLS calls with `between(s, P, k)` after each but the last; nothing reads the state before the end."""
    import torch
    import paper_2606_12850_amd as P
    mesh = W.box_mesh(4, N, 4000.0, jitter=0.1, seed=3)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        s = P.Solver(N)
        s.upload_mesh(mesh)
        s.upload_model(*W.layered_model(mesh, grf_amp=0.05, grf_seed=1))
        P.semx_set_geometry(s.ctx, P.SEMX_GEOM_TRILINEAR)  # the element blocks run only where they are switched on
        dt = 0.5 * P.semx_cfl_dt(s.ctx, 0.4)
        nt = CALLS * STEPS
        f0 = 0.25 / (20 * dt)
        s.stf = (W.ricker(f0, 1.2 / f0, dt, nt + 1)[None, :] * 1e9).astype(np.float32)
        s.src = W.center_vertex_source(mesh)
        re, rx = W.top_receivers_line(mesh, 6)
        P.semx_set_sources(s.ctx, *s.src, np.array([[0.3, -0.2, 1.0]]), s.stf)
        P.semx_set_receivers(s.ctx, re, rx, nt)
        s.nrec, s.nt_max = len(re), nt
        P.semx_set_dt(s.ctx, dt)
        P.semx_reset(s.ctx)
        P.semx_set_graphs(s.ctx, chunk)
        s.ug = torch.full((mesh.nglob, 3), 1.0, device="cuda")
        s.ug += torch.arange(mesh.nglob, device="cuda")[:, None] * 1e-3
        s.fg = s.empty_field()
        s.side = side
        for k in range(CALLS):
            s.step(STEPS)
            if k + 1 < CALLS and between is not None:
                between(s, P, k)
        u, v = s.empty_field(), s.empty_field()
        P.semx_get_state(s.ctx, u, v)
        side.synchronize()
        out = u.cpu().numpy(), v.cpu().numpy(), s.seismograms()
    s.close()
    assert all(np.abs(x).max() > 0 for x in out)
    return out


def _apply(s, P, k):
    s.apply_force(s.ug, s.fg)


def _sources(s, P, k):
    P.semx_set_sources(s.ctx, *s.src, np.array([[0.1 * k, 1.0, 0.5]]), s.stf)


def _eigen(s, P, k):
    P.semx_max_eigenvalue(s.ctx, 1)


def _skeleton(s, P, k):
    P.semx_force_skeleton(s.ctx, s.ug, s.fg, 1)


def _blocks(s, P, k):
    P.semx_set_blocks(s.ctx, P.SEMX_BLOCKS_OFF if k % 2 else P.SEMX_BLOCKS_ON)


def _assembly(s, P, k):
    s.set_mode(P.SEMX_C_F32, P.SEMX_ASM_COLORED if k % 2 else P.SEMX_ASM_ATOMIC)


@pytest.mark.parametrize("between", [None, _apply, _sources, _eigen, _skeleton, _blocks],
                         ids=["nothing", "apply", "sources", "eigenvalue", "skeleton", "blocks"])
def test_graphs_bitwise(between):
    for x, y in zip(_run(between, 0), _run(between, CHUNK)):
        np.testing.assert_array_equal(x, y)


def test_graphs_assembly_switched():
    """Atomic segments add in hardware order: FP32 rounding grown over the steps, as in the graph tests."""
    for x, y in zip(_run(_assembly, 0), _run(_assembly, CHUNK)):
        assert rel_l2(y, x) <= 1e-5


@pytest.mark.parametrize("between", [_apply, _eigen, _skeleton], ids=["apply", "eigenvalue", "skeleton"])
@pytest.mark.parametrize("chunk", [0, CHUNK])
def test_applies_leave_the_run(between, chunk):
    for x, y in zip(_run(None, 0), _run(between, chunk)):
        np.testing.assert_array_equal(x, y)


def _capture(s):
    """A graph of one apply; the pending force is that of the step before it."""
    import torch
    g = torch.cuda.CUDAGraph()
    s.side.synchronize()
    with torch.cuda.graph(g, stream=s.side):
        s.apply_force(s.ug, s.fg)
    return g


def test_replayed_applies_leave_the_run():
    """A caller's graph of an apply, captured between two calls and replayed after later ones."""
    got = {}

    def between(s, P, k):
        if k == 0:
            s.apply_force(s.ug, s.fg)
            got["eager"] = s.fg.cpu().numpy()
            got["graph"] = _capture(s)
        s.fg.zero_()
        for _ in range(2):
            got["graph"].replay()
        s.side.synchronize()
        np.testing.assert_array_equal(s.fg.cpu().numpy(), got["eager"])

    def captured_only(s, P, k):
        got["unused"] = _capture(s)  # captured, never replayed

    plain = _run(None, 0)
    for fn in (between, captured_only):
        for x, y in zip(plain, _run(fn, 0)):
            np.testing.assert_array_equal(x, y)


def _captured_first_apply(f64):
    """On a caller's colouring, the first force pass of all is recorded into a graph."""
    import torch
    import paper_2606_12850_amd as P
    mesh = W.box_mesh((3, 2, 3), N, 4000.0, jitter=0.1, seed=4)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        s = P.Solver(N, storage=P.SEMX_F64 if f64 else P.SEMX_F32)
        s.upload_mesh(mesh)
        P.semx_set_coloring(s.ctx, *P.semx_get_coloring(s.ctx, mesh.nspec))
        s.upload_model(*W.layered_model(mesh))
        s.ug, s.fg, s.side = s.empty_field(), s.empty_field(), side
        s.ug += torch.arange(mesh.nglob, device="cuda")[:, None] * 1e-3
        s.ug *= s.ug
        g = _capture(s)
        s.fg.fill_(1.0)
        g.replay()
        first = s.fg.clone()
        s.apply_force(s.ug, s.fg)
        side.synchronize()
        out = first.cpu().numpy(), s.fg.cpu().numpy()
    s.close()
    return out


@pytest.mark.parametrize("f64", [False, True], ids=["f32", "f64"])
def test_first_pass_captured(f64):
    graph, direct = _captured_first_apply(f64)
    assert np.abs(direct).max() > 0
    np.testing.assert_array_equal(graph, direct)
