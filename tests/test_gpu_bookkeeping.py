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

pytestmark = pytest.mark.gpu


def _pass_us(n, ne, nsrc, nrec, acoustic, f64=False, steps=60):
    import paper_2606_12850_amd as P
    mesh = W.box_mesh(ne, n, 4000.0)
    s = P.Solver(n, physics=P.SEMX_ACOUSTIC if acoustic else P.SEMX_ELASTIC,
                 storage=P.SEMX_F64 if f64 else P.SEMX_F32)
    s.upload_mesh(mesh)
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
