"""The time loop's bookkeeping (receivers, source work) does not hold up the force launch that carries it.

The waves of a force launch that record receivers and sum the source work end
before its elements do; where they would not (many receiver or source points for
the elements' time) they have a launch of their own.  The force pass's own time,
from the library's events, is therefore that of a loop without any, within the
spread of two timings and an event's resolution.
"""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import rel_l2

pytestmark = pytest.mark.gpu


def _solver(n, ne, nsrc, nrec, acoustic, f64, steps, own_colors=False):
    import paper_2606_12850_amd as P
    mesh = W.box_mesh(ne, n, 4000.0)
    s = P.Solver(n, physics=P.SEMX_ACOUSTIC if acoustic else P.SEMX_ELASTIC,
                 storage=P.SEMX_F64 if f64 else P.SEMX_F32)
    s.upload_mesh(mesh)
    if own_colors:
        P.semx_set_coloring(s.ctx, *P.semx_get_coloring(s.ctx, mesh.nspec))
    lam, mu, rho = W.homogeneous_model(mesh)
    if acoustic:
        s.upload_model_acoustic(lam, rho)
    else:
        s.upload_model(lam, mu, rho)
    rng = np.random.default_rng(0)
    if nsrc:
        stf = rng.standard_normal((nsrc, steps + 2)) * 1e9
        el, xi = rng.integers(0, mesh.nspec, nsrc).astype(np.int32), rng.uniform(-0.9, 0.9, (nsrc, 3))
        d = None if acoustic else rng.standard_normal((nsrc, 3))
        if f64:
            P.semx_set_sources_f64(s.ctx, el, xi, d, stf)
        else:
            P.semx_set_sources(s.ctx, el, xi, d, stf.astype(np.float32))
    if nrec:
        P.semx_set_receivers(s.ctx, rng.integers(0, mesh.nspec, nrec).astype(np.int32),
                             rng.uniform(-0.9, 0.9, (nrec, 3)), steps)
        s.nrec, s.nt_max = nrec, steps
    P.semx_set_dt(s.ctx, P.semx_cfl_dt(s.ctx, 0.3))
    return P, s


def _pass_us(n, ne, nsrc, nrec, acoustic, steps=60):
    P, s = _solver(n, ne, nsrc, nrec, acoustic, False, steps)
    best = np.inf
    for _ in range(4):
        P.semx_reset(s.ctx)
        P.semx_set_timing(s.ctx, 1)
        s.step(steps)
        launches, ms = P.semx_force_timing(s.ctx)
        best = min(best, ms / launches * 1e3)
    s.close()
    return best


@pytest.mark.parametrize("n,ne,nsrc,nrec,acoustic", [
    (16, 2, 1, 8, False), (16, (102, 1, 1), 1, 1, True), (14, 1, 1, 4, False),
])
def test_receivers_of_the_high_orders(n, ne, nsrc, nrec, acoustic):
    alone, loaded = _pass_us(n, ne, 0, 0, acoustic), _pass_us(n, ne, nsrc, nrec, acoustic)
    print(f"force launch {alone:.1f} us, with bookkeeping {loaded:.1f} us")
    assert loaded <= 1.25 * alone + 3.0


@pytest.mark.parametrize("n,ne,nsrc,acoustic", [
    (5, 4, 64, False), (5, 4, 64, True), (5, 12, 256, False), (8, 8, 32, False), (12, 3, 8, False),
])
def test_work_of_many_sources(n, ne, nsrc, acoustic):
    alone, loaded = _pass_us(n, ne, 0, 0, acoustic), _pass_us(n, ne, nsrc, 4, acoustic)
    print(f"force launch {alone:.1f} us, with bookkeeping {loaded:.1f} us")
    assert loaded <= 1.25 * alone + 3.0


@pytest.mark.parametrize("n,ne,nsrc,acoustic,f64", [
    (5, 4, 64, False, False), (9, 2, 8, False, False), (5, 3, 64, True, False),
    (5, 4, 64, False, True), (9, 2, 8, False, True),
])
def test_many_sources_as_colour_by_colour(n, ne, nsrc, acoustic, f64):
    """Seismograms, energy and source work as with the pass colour by colour: to the bit in FP32, in FP64 (where that
    pass adds the source force after the elements' forces, not before) to its rounding: 30 steps of 9 terms, 3e-14."""
    out = []
    for own_colors in (False, True):
        P, s = _solver(n, ne, nsrc, 5, acoustic, f64, 30, own_colors)
        P.semx_reset(s.ctx)
        s.step(17)
        s.step(13)
        out.append((s.seismograms(), P.semx_energy(s.ctx)))
        s.close()
    if f64:
        assert rel_l2(out[0][0], out[1][0]) < 1e-12
        assert np.allclose(out[0][1], out[1][1], rtol=1e-12, atol=0)
    else:
        assert np.array_equal(out[0][0], out[1][0])
        assert out[0][1] == out[1][1]
