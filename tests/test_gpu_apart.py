"""Force applies on elements that touch nowhere, at the orders and sizes whose
ordinary passes run on the line kernel: one launch that stores into f, to the bit
the pass colour by colour, up to the size where the line kernel and a nodal sum
are faster (then to rounding).
"""
from types import SimpleNamespace

import numpy as np
import pytest

import workloads as W
from tests.gpu_common import rel_l2

pytestmark = pytest.mark.gpu

# NGLL, elements, acoustic, direct
CASES = [(2, 1, False, True), (2, 1, True, True), (2, 300, False, True), (2, 16500, False, False), (3, 9800, False, True),
         (8, 520, False, True), (8, 520, True, True), (11, 2, False, False), (12, 1, False, True), (12, 3, True, True),
         (12, 620, False, False)]


@pytest.mark.parametrize("n,elements,acoustic,direct", CASES)
def test_apply(n, elements, acoustic, direct):
    import torch
    import paper_2606_12850_amd as P
    one = W.box_mesh((1, 1, 1), n, 1000.0)
    k = np.arange(elements)[:, None]
    at = np.stack([2000.0 * (k[:, 0] % 100), 2000.0 * (k[:, 0] // 100), 0.0 * k[:, 0]], axis=-1)
    mesh = SimpleNamespace(n=n, nspec=elements, nglob=elements * one.nglob,
                           ibool=(one.ibool + k * one.nglob).astype(np.int32),
                           elem_vert=(one.elem_vert + k * len(one.vert)).astype(np.int32),
                           vert=(at[:, None] + one.vert).reshape(-1, 3))
    rng = np.random.default_rng(n)
    lam = rng.uniform(1e9, 2e9, (elements, n ** 3))
    u = torch.from_numpy(rng.uniform(-1, 1, (mesh.nglob,) if acoustic else (mesh.nglob, 3)).astype(np.float32)).cuda()
    out = []
    for own in (False, True):
        s = P.Solver(n, physics=P.SEMX_ACOUSTIC if acoustic else P.SEMX_ELASTIC)
        s.upload_mesh(mesh)
        if own:
            P.semx_set_coloring(s.ctx, *P.semx_get_coloring(s.ctx, elements))
        (s.upload_model_acoustic(lam, np.full_like(lam, 1000.0)) if acoustic
         else s.upload_model(lam, 0.5 * lam, np.full_like(lam, 2500.0)))
        f = torch.full_like(u, 7.0)
        s.apply_force(u, f)
        torch.cuda.synchronize()
        out.append(f.cpu().numpy())
        s.close()
    assert np.abs(out[1]).max() > 0
    if direct:
        np.testing.assert_array_equal(*out)
    else:
        # two FP32 sums of 6 n + 30 roundings of 6e-8, with the row sums of |D| up to 100 at NGLL 12 as amplification
        assert rel_l2(*out) <= 6e-8 * np.sqrt(6 * n + 30) * 100
