"""Elements around an axis: nodes that many elements share (the sort of their
points goes through a heap from 33 on), against the FP64 oracle and, to the bit,
against the pass colour by colour.
"""
from types import SimpleNamespace

import numpy as np
import pytest

from tests.gpu_common import oracle_geometry, rel_l2

pytestmark = pytest.mark.gpu


def _fan(sectors, layers, n):
    """Kites around the z axis: corners axis, ray k, outer point, ray k + 1."""
    import paper_2606_12850_amd as P
    t = 2 * np.pi * np.arange(sectors) / sectors
    vert, ev = [], []
    for z in range(layers + 1):
        base = z * (2 * sectors + 1)
        vert += [[0.0, 0.0, 100.0 * z]]
        vert += [[100 * np.cos(a), 100 * np.sin(a), 100.0 * z] for a in t]
        vert += [[130 * np.cos(a + np.pi / sectors), 130 * np.sin(a + np.pi / sectors), 100.0 * z] for a in t]
        if z == layers:
            continue
        up = 2 * sectors + 1
        for k in range(sectors):
            low = [base, base + 1 + k, base + 1 + (k + 1) % sectors, base + 1 + sectors + k]
            ev.append(low + [v + up for v in low])
    vert, ev = np.array(vert), np.array(ev, np.int32)
    xi = np.array(P.semx_gll(n)[0])
    k, j, i = (q.ravel() for q in np.meshgrid(xi, xi, xi, indexing="ij"))
    shape = [(1 + (1 if v & 1 else -1) * i) * (1 + (1 if v & 2 else -1) * j) * (1 + (1 if v & 4 else -1) * k) / 8
             for v in range(8)]
    xyz = np.einsum("evc,vq->eqc", vert[ev], np.array(shape)).reshape(-1, 3)
    _, ibool = np.unique(np.round(xyz, 6) + 0.0, axis=0, return_inverse=True)
    ibool = ibool.reshape(len(ev), n ** 3).astype(np.int32)
    return SimpleNamespace(n=n, nspec=len(ev), nglob=int(ibool.max()) + 1, ibool=ibool, vert=vert, elem_vert=ev)


@pytest.mark.parametrize("sectors,layers,n", [(32, 1, 4), (33, 1, 3), (48, 2, 5), (150, 1, 2)])
def test_shared_axis(orc, sectors, layers, n):
    import torch
    import paper_2606_12850_amd as P
    m = _fan(sectors, layers, n)
    assert np.bincount(m.ibool.ravel()).max() >= sectors
    rng = np.random.default_rng(sectors)
    r = rng.uniform(0.9, 1.1, (m.nspec, n ** 3))
    lam, mu, rho = 2.0e10 * r, 1.0e10 * r, np.full_like(r, 2500.0)
    u = rng.uniform(-1, 1, (m.nglob, 3)).astype(np.float32)
    out = []
    for own in (False, True):
        s = P.Solver(n)
        s.upload_mesh(m)
        if own:
            P.semx_set_coloring(s.ctx, *P.semx_get_coloring(s.ctx, m.nspec))
        s.upload_model(lam, mu, rho)
        P.semx_set_checkpointing(s.ctx, 100)  # the same element kernels on both routes
        out.append(s.apply_force(torch.from_numpy(u).cuda()).cpu().numpy())
        s.close()
    np.testing.assert_array_equal(*out)
    gam, jac, _ = oracle_geometry(orc, m)
    # FP32 sums of up to 150 elements' forces, each of some 6 n + 30 roundings of 6e-8, amplified by the kites' aspect
    # ratio (up to 20) in Gamma
    assert rel_l2(out[0], orc.force(n, m.ibool, gam, jac, lam, mu, u.astype(np.float64), m.nglob)) <= 5e-5
