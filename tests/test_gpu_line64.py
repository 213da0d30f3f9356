"""The line kernel in double (from 2^17 points with one Gamma per element, from
2^18 points at NGLL 6 and more with Gamma at each point) against the FP64 oracle.
"""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import oracle_geometry, rel_l2
from tests.test_gpu_fp64 import gpu_force64, solver64

pytestmark = pytest.mark.gpu

# two FP64 evaluations of one sum of some 12 n + 60 roundings of 1.1e-16, amplified by the cancellation of the
# derivatives (row sums of |D| up to 80 at NGLL 10): 1e-16 x sqrt(180) x 80 = 1e-13, with a margin of ten for the
# rounding of the vertex coordinates, which regular elements take from one point for all
TOL = 1e-12

EXTENTS = {2: (33, 25, 21), 3: (19, 17, 16), 4: (13, 13, 13), 5: (11, 10, 10), 6: (9, 9, 8), 7: (8, 7, 7),
           8: (7, 7, 6), 9: (6, 6, 5), 10: (6, 5, 5)}
STORED = {6: (11, 11, 11), 7: (10, 9, 9), 8: (9, 8, 8), 9: (8, 7, 7), 10: (7, 7, 6)}
CASES = [(n, ne, k) for n, ne in EXTENTS.items() for k in ("regular", "scrambled")]
CASES += [(n, ne, "jittered") for n, ne in STORED.items()] + [(7, STORED[7], "offset")]


@pytest.mark.parametrize("n,ne,kind", CASES)
def test_line64_force(orc, n, ne, kind):
    m = W.box_mesh(ne, n, tuple(100.0 * x for x in ne), jitter=0.1 if kind == "jittered" else 0.0, seed=n)
    if kind == "scrambled":
        m.ibool = np.random.default_rng(9).permutation(m.nglob).astype(np.int32)[m.ibool]
    if kind == "offset":  # nearly affine: one corner off by 4e-13 of an edge, more than its coordinates round by
        m.vert[m.elem_vert[0, 0]] -= 4e-11
    rng = np.random.default_rng(n)
    r = rng.uniform(0.8, 1.2, (m.nspec, n ** 3))
    lam, mu, rho = 2.0e10 * r, 1.0e10 * r[::-1], np.full_like(r, 2500.0)
    gam, jac, _ = oracle_geometry(orc, m)
    u = rng.uniform(-1, 1, (m.nglob, 3))
    s = solver64(n)
    s.upload_mesh(m)
    s.upload_model(lam, mu, rho)
    f = gpu_force64(s, u)
    assert np.array_equal(f, gpu_force64(s, u))
    s.close()
    err = rel_l2(f, orc.force(n, m.ibool, gam, jac, lam, mu, u, m.nglob))
    print(f"line64 n={n} {ne} {kind}: {err:.2e}")
    assert err <= TOL
