"""The line kernel (one lane per line of points, NGLL 2-12) against the FP64
oracle.

It runs where a pass fills the chip (2^18 points and more; at NGLL 2, 11 and
12 at any size), several elements to a workgroup: the meshes here end in
groups that are not full, have odd extents, and one whose node numbers are no
lattice.
"""
import numpy as np
import pytest

import workloads as W
from oracle import acoustic as A
from tests.gpu_common import gpu_force, make_solver, oracle_geometry, rel_l2

pytestmark = pytest.mark.gpu

# FP32 against FP64: the largest of the about 12 n + 60 roundings of 2^-24 that a point's force passes through,
# amplified by the cancellation of a derivative (row sums of |D| up to 120 at NGLL 12 against results of order one)
# and averaged over the field: the bar of the other FP32 force tests
TOL = 1e-5

EXTENTS = {3: (31, 20, 17), 4: (17, 16, 17), 5: (13, 13, 13), 6: (12, 11, 10), 7: (9, 10, 9), 8: (9, 8, 8),
           9: (8, 8, 6), 10: (7, 6, 7)}
CASES = [(n, ne, kind, geo) for n, ne in EXTENTS.items()
         for kind, geo in (("regular", 0), ("jittered", 1), ("scrambled", 1), ("jittered", 0)) if geo or n > 5 or kind != "jittered"]
CASES += [(n, ne, kind, geo) for n in (2, 11, 12) for ne in ((1, 1, 1), (3, 2, 3)) for kind, geo in
          (("regular", 0), ("jittered", 0), ("jittered", 1), ("scrambled", 1))]
CASES += [(2, (33, 5, 7), "jittered", 1)]


def _mesh(n, ne, kind):
    m = W.box_mesh(ne, n, tuple(100.0 * x for x in ne), jitter=0.0 if kind == "regular" else 0.1, seed=n)
    if kind == "jittered" and ne == (1, 1, 1):  # no interior vertex: move a corner
        m.vert[-1] += (5.0, -4.0, 6.0)
    if kind == "scrambled":
        m.ibool = np.random.default_rng(9).permutation(m.nglob).astype(np.int32)[m.ibool]
    return m


@pytest.mark.parametrize("n,ne,kind,geo", CASES)
def test_line_force(orc, n, ne, kind, geo):
    import paper_2606_12850_amd as P
    m = _mesh(n, ne, kind)
    rng = np.random.default_rng(n)
    r = rng.uniform(0.8, 1.2, (m.nspec, n ** 3))
    lam, mu, rho = 2.0e10 * r, 1.0e10 * r[::-1], np.full_like(r, 2500.0)
    gam, jac, _ = oracle_geometry(orc, m)
    u = rng.uniform(-1, 1, (m.nglob, 3)).astype(np.float32).astype(np.float64)
    s = make_solver(n)
    s.upload_mesh(m)
    P.semx_set_geometry(s.ctx, geo)
    P.semx_set_blocks(s.ctx, P.SEMX_BLOCKS_OFF)
    s.upload_model(lam, mu, rho)
    f = gpu_force(s, u)
    assert np.array_equal(f, gpu_force(s, u))
    err = rel_l2(f, orc.force(n, m.ibool, gam, jac, lam, mu, u, m.nglob))
    s.close()
    print(f"line n={n} {ne} {kind} geometry {geo}: {err:.2e}")
    assert err <= TOL
    a = P.Solver(n, physics=P.SEMX_ACOUSTIC)
    a.upload_mesh(m)
    P.semx_set_geometry(a.ctx, geo)
    a.upload_model_acoustic(2.25e9 * r, 1000.0 * r[::-1])
    err = rel_l2(gpu_force(a, u[:, 0]), A.force(n, m.ibool, gam, jac, 1000.0 * r[::-1], u[:, 0], m.nglob))
    a.close()
    print(f"line n={n} {ne} {kind} geometry {geo} acoustic: {err:.2e}")
    assert err <= TOL


def test_line_batched_models(orc):
    """Two models on one mesh, together past the line kernel's size."""
    import paper_2606_12850_amd as P
    n, m = 5, _mesh(5, (11, 10, 11), "regular")
    rng = np.random.default_rng(1)
    r = rng.uniform(0.8, 1.2, (2, m.nspec, n ** 3))
    lam, mu, rho = 2.0e10 * r, 1.0e10 * r, np.full_like(r, 2500.0)
    gam, jac, _ = oracle_geometry(orc, m)
    u = rng.uniform(-1, 1, (2, m.nglob, 3)).astype(np.float32).astype(np.float64)
    s = make_solver(n)
    s.upload_mesh(m)
    s.upload_model(lam, mu, rho)
    f = gpu_force(s, u)
    s.close()
    for k in range(2):
        assert rel_l2(f[k], orc.force(n, m.ibool, gam, jac, lam[k], mu[k], u[k], m.nglob)) <= TOL
