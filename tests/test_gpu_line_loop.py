"""Time loops on the line kernel: the bookkeeping waves that ride in its launch
(receivers, source work, the coming source force), split launches of affine and
other numberings, and graph-captured steps.
"""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_assembly import _mesh, _run

pytestmark = pytest.mark.gpu

# above 2^17 points with one Gamma per element, above 2^18 with Gamma at each; a periodic box has elements with and
# without an affine numbering
FP64 = [(5, (11, 10, 10), "regular"), (5, (11, 10, 10), "scrambled"), (4, (13, 13, 13), "periodic"),
        (7, (10, 9, 9), "jittered"), (10, (6, 5, 5), "regular")]

# a force of the two kernels agrees to 1e-13 (roundings of 1.1e-16, amplified by the row sums of |D|); 24 steps of a
# recursion that preserves a difference, and the forces of a difference that the step's stability bounds
TOL = 24 * 2 * 1e-13


@pytest.mark.parametrize("n,ne,kind", FP64)
def test_fp64_loop(n, ne, kind):
    import paper_2606_12850_amd as P
    mesh = _mesh(kind, n, ne)
    for a, b in zip(_run(P, mesh, n, False, 0, storage=P.SEMX_F64), _run(P, mesh, n, True, 0, storage=P.SEMX_F64)):
        assert np.abs(b).max() > 0
        assert np.linalg.norm(a - b) <= TOL * np.linalg.norm(b)


def _graph_run(n, ne, kind, chunk):
    import torch
    import paper_2606_12850_amd as P
    mesh = _mesh(kind, n, ne)
    s = P.Solver(n)
    s.upload_mesh(mesh)
    P.semx_set_geometry(s.ctx, P.SEMX_GEOM_TRILINEAR)
    s.upload_model(*W.homogeneous_model(mesh))
    nt = 60
    se, sx = np.array([0, mesh.nspec // 2], np.int32), np.array([[1.0, 1.0, 1.0], [0.2, -0.4, 0.6]])
    stf = 1e9 * np.random.default_rng(5).uniform(-1, 1, (2, nt + 1)).astype(np.float32)
    P.semx_set_sources(s.ctx, se, sx, np.array([[0.0, 0.0, 1.0], [1.0, 0.5, 0.0]]), stf)
    P.semx_set_receivers(s.ctx, se, sx, nt)
    s.nrec, s.nt_max = 2, nt
    P.semx_set_dt(s.ctx, P.semx_cfl_dt(s.ctx, 0.3))
    P.semx_reset(s.ctx)
    P.semx_set_graphs(s.ctx, chunk)
    out = []
    for k in (25, 3, 30):
        s.step(k)
        out.append(np.array(P.semx_energy(s.ctx, True)))
    u, v = s.empty_field(), s.empty_field()
    P.semx_get_state(s.ctx, u, v)
    torch.cuda.synchronize()
    out += [u.cpu().numpy(), v.cpu().numpy(), s.seismograms()]
    s.close()
    return out


@pytest.mark.parametrize("n,ne,kind", [(2, (5, 4, 3), "mixed"), (5, (15, 13, 12), "regular"), (11, (2, 1, 2), "jittered"),
                                       (12, (3, 2, 2), "periodic")])
def test_graph_steps(n, ne, kind):
    for a, b in zip(_graph_run(n, ne, kind, 0), _graph_run(n, ne, kind, 8)):
        assert np.abs(a).max() > 0
        np.testing.assert_array_equal(a, b)
