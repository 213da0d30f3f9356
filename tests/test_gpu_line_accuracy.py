"""The line kernel's forces are as near to FP64 as the per-point kernels'.

Both kernels on the same mesh, model and field (the per-point ones through a
colouring of the caller's) against the FP64 storage of the library.
"""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import rel_l2

pytestmark = pytest.mark.gpu


def _field(mesh, rng):
    """Cosines of 5 to 30 nodes per wavelength along each axis of the node lattice."""
    g = mesh.lattice_index()
    u = np.zeros((mesh.nglob, 3))
    for c in range(3):
        w = np.zeros(mesh.ibool.shape)
        for _ in range(3):
            w += np.prod([np.cos(2 * np.pi / rng.uniform(5, 30) * x + rng.uniform(0, 6.3)) for x in g], axis=0)
        u[mesh.ibool.ravel(), c] = w.ravel()
    return u.astype(np.float32)


def _forces(mesh, model, u, trilinear, own_colours=False, f64=False):
    import torch
    import paper_2606_12850_amd as P
    s = P.Solver(mesh.n, storage=P.SEMX_F64 if f64 else P.SEMX_F32)
    s.upload_mesh(mesh)
    if own_colours:
        P.semx_set_coloring(s.ctx, *P.semx_get_coloring(s.ctx, mesh.nspec))
    if trilinear and not f64:
        P.semx_set_geometry(s.ctx, P.SEMX_GEOM_TRILINEAR)
    s.upload_model(*model)
    f = s.apply_force(torch.from_numpy(u).to("cuda", torch.float64 if f64 else torch.float32))
    torch.cuda.synchronize()
    s.close()
    return f.cpu().numpy()


# The two errors are norms over 1e5 and more roundings of one size, so their ratio is 1 to a few per cent; runs of
# equal roundings (one field's symmetries) may add a few more.
RATIO = 1.1


@pytest.mark.parametrize("trilinear", [False, True], ids=["regular", "trilinear"])
@pytest.mark.parametrize("n", range(2, 11))
def test_error_against_fp64(n, trilinear):
    side = int(np.ceil(2 ** 6 / n)) + 1  # above 2^18 points
    line, point = [], []
    for seed in range(4):
        mesh = W.box_mesh((side, side, side + 1), n, 4000.0, jitter=0.1 if trilinear else 0.0, seed=seed)
        rng = np.random.default_rng(seed)
        model = W.layered_model(mesh, grf_amp=0.05, grf_seed=seed)
        u = _field(mesh, rng)
        ref = _forces(mesh, model, u, trilinear, f64=True)
        line.append(rel_l2(_forces(mesh, model, u, trilinear), ref))
        point.append(rel_l2(_forces(mesh, model, u, trilinear, own_colours=True), ref))
    print(f"n={n} line {np.mean(line):.2e}, one lane per point {np.mean(point):.2e}")
    assert np.mean(line) <= RATIO * np.mean(point)
