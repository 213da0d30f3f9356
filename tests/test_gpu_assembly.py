"""The assembly through element-local forces and nodal sums against the pass
colour by colour.

Giving the library its own colouring back (semx_set_coloring) makes it run
colour by colour, one launch per colour with read-modify-write.  Without it
the force is one launch over the mesh and a sum per node, in the order in
which the coloured pass reaches the node: the same additions, so the FP32
results agree to the bit, and so do the time loops (whose Newmark pass sums
the node's points itself).  Elastic FP32 runs are made with checkpoints on:
those keep the element kernels of the coloured pass at every size.
"""
from types import SimpleNamespace

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _model(mesh, seed, acoustic):
    r = np.random.default_rng(seed).uniform(0.9, 1.1, (mesh.nspec, mesh.n ** 3))
    lam, mu = W.lame(3000.0 * r, 1732.0 * r, 2500.0)
    return (lam, np.full_like(lam, 1000.0)) if acoustic else (lam, mu, np.full_like(lam, 2500.0))


def _mesh(kind, n, ne):
    if kind == "periodic":
        return W.box_mesh(ne, n, 1000.0, periodic=True)
    m = W.box_mesh(ne, n, 1000.0, jitter=0.1 if kind in ("jittered", "scrambled", "mixed") else 0.0, seed=4)
    if kind == "scrambled":  # no lattice: any node order
        m.ibool = np.random.default_rng(2).permutation(m.nglob).astype(np.int32)[m.ibool]
    if kind == "mixed":  # regular and irregular elements side by side
        v = W.box_mesh(ne, n, 1000.0).vert
        keep = v[:, 0] > 500.0
        m.vert[keep] = v[keep]
    return m


def _run(P, mesh, n, colours, geometry, mode=None, storage=0, acoustic=False, models=1):
    import torch
    s = P.Solver(n, storage=storage, physics=P.SEMX_ACOUSTIC if acoustic else P.SEMX_ELASTIC)
    s.upload_mesh(mesh)
    if colours:
        P.semx_set_coloring(s.ctx, *P.semx_get_coloring(s.ctx, mesh.nspec))
    P.semx_set_blocks(s.ctx, P.SEMX_BLOCKS_OFF)
    P.semx_set_geometry(s.ctx, geometry)
    model = [_model(mesh, k, acoustic) for k in range(models)]
    model = model[0] if models == 1 else [np.stack(m) for m in zip(*model)]
    (s.upload_model_acoustic if acoustic else s.upload_model)(*model)
    if mode is not None:
        s.set_mode(mode)
    f64 = storage == P.SEMX_F64
    if not f64 and not acoustic:
        P.semx_set_checkpointing(s.ctx, 6)
    u = s.empty_field()
    u.copy_(torch.from_numpy(np.random.default_rng(3).uniform(-1, 1, tuple(u.shape))))
    out = [s.apply_force(u).cpu().numpy()]
    se, sx = np.array([0, mesh.nspec // 2], np.int32), np.array([[1.0, 1.0, 1.0], [0.2, -0.4, 0.6]])
    sd = None if acoustic else np.array([[0.0, 0.0, 1.0], [1.0, 0.5, 0.0]])
    stf = np.random.default_rng(5).uniform(-1, 1, (2, 32))
    (P.semx_set_sources_f64 if f64 else P.semx_set_sources)(s.ctx, se, sx, sd, stf)
    P.semx_set_receivers(s.ctx, se, np.array([[0.1, 0.2, 0.3], [1.0, -1.0, 0.0]]), 30)
    s.nrec, s.nt_max = 2, 30
    P.semx_set_dt(s.ctx, P.semx_cfl_dt(s.ctx, 0.3))
    P.semx_reset(s.ctx)
    P.semx_step(s.ctx, 7)
    P.semx_step(s.ctx, 1)
    out.append(s.apply_force(u).cpu().numpy())  # between steps: the pending force is kept
    P.semx_step(s.ctx, 5)
    # other sources from here on: the pending force keeps the old ones
    (P.semx_set_sources_f64 if f64 else P.semx_set_sources)(s.ctx, se[:1], sx[:1], sd if sd is None else sd[:1], stf[1:])
    P.semx_step(s.ctx, 9)
    uu, vv, aa = (s.empty_field() for _ in range(3))
    (P.semx_get_state_f64 if f64 else P.semx_get_state)(s.ctx, uu, vv, aa)
    P.semx_step(s.ctx, 2)
    out += [t.cpu().numpy() for t in (uu, vv, aa)] + [s.seismograms(), np.array(P.semx_energy(s.ctx, True))]
    s.close()
    return out


CASES = [  # n, elements, mesh, geometry (0 stored, 1 trilinear), mode, physics and storage
    *((n, (3, 2, 3), "jittered", n % 2, None, "elastic") for n in range(2, 13)),
    *((n, (2, 2, 3), "regular", 0, None, "elastic") for n in (2, 5, 8, 12, 13, 16)),
    (5, (1, 1, 1), "regular", 0, None, "elastic"), (4, (1, 7, 1), "regular", 0, None, "elastic"),
    (3, (40, 3, 2), "jittered", 0, None, "elastic"), (6, (4, 4, 4), "scrambled", 0, None, "elastic"),
    (5, (4, 4, 3), "mixed", 0, None, "elastic"), (5, (4, 3, 3), "mixed", 1, None, "elastic"),
    (4, (4, 4, 5), "periodic", 0, None, "elastic"), (16, (2, 1, 2), "scrambled", 0, None, "elastic"),
    (5, (3, 4, 2), "jittered", 0, "bf16", "elastic"), (8, (2, 3, 2), "regular", 0, "f16", "elastic"),
    (12, (2, 3, 2), "regular", 0, "bf16", "elastic"), (14, (2, 1, 2), "jittered", 1, "f16", "elastic"),
    *((n, (3, 2, 2), "jittered", n % 2, None, "acoustic") for n in (3, 5, 10, 13, 16)),
    (8, (19, 1, 1), "regular", 0, None, "acoustic"), (5, (4, 5, 3), "scrambled", 0, None, "acoustic"),
    *((n, (3, 2, 2), "jittered", 0, None, "f64") for n in (2, 5, 10)), (4, (4, 4, 4), "scrambled", 0, None, "f64"),
]


@pytest.mark.parametrize("n,ne,kind,geometry,mode,what", CASES)
def test_nodal_sums_equal_coloured_pass(n, ne, kind, geometry, mode, what):
    import paper_2606_12850_amd as P
    mesh = _mesh(kind, n, ne)
    kw = {"geometry": geometry, "mode": {None: None, "bf16": P.SEMX_C_BF16, "f16": P.SEMX_C_F16}[mode],
          "storage": P.SEMX_F64 if what == "f64" else P.SEMX_F32, "acoustic": what == "acoustic"}
    for a, b in zip(_run(P, mesh, n, False, **kw), _run(P, mesh, n, True, **kw)):
        if what == "f64":
            # the coloured pass adds the source after the elements, the sum starts from it: a few roundings of 1e-16
            # a step apart, over 24 steps
            assert np.linalg.norm(a - b) <= 1e-13 * np.linalg.norm(b)
        else:
            np.testing.assert_array_equal(a, b)


def test_nodal_sums_batched_models():
    import paper_2606_12850_amd as P
    mesh = _mesh("regular", 5, (3, 2, 4))
    for a, b in zip(_run(P, mesh, 5, False, 0, models=3), _run(P, mesh, 5, True, 0, models=3)):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("n,ne,kind,geometry", [(5, (3, 2, 3), "regular", 0), (4, (3, 3, 3), "scrambled", 1),
                                                (5, (4, 3, 2), "mixed", 0), (2, (9, 4, 5), "jittered", 1),
                                                (12, (2, 2, 1), "jittered", 0)])
def test_adjoint_on_nodal_sums(n, ne, kind, geometry):
    """Gradients through element-local forces and nodal sums against the pass
    colour by colour; receivers that share nodes, one of them on a node."""
    import torch
    import paper_2606_12850_amd as P
    mesh, out = _mesh(kind, n, ne), []
    for colours in (False, True):
        s = P.Solver(n)
        s.upload_mesh(mesh)
        if colours:
            P.semx_set_coloring(s.ctx, *P.semx_get_coloring(s.ctx, mesh.nspec))
        P.semx_set_geometry(s.ctx, geometry)
        P.semx_set_blocks(s.ctx, P.SEMX_BLOCKS_OFF)
        s.upload_model(*_model(mesh, 1, False))
        el = np.array([0, 1, 1, mesh.nspec - 1], np.int32)
        P.semx_set_sources(s.ctx, el[1:2], np.array([[0.3, -0.2, 0.1]]), np.array([[1.0, 0.4, -0.7]]),
                           np.random.default_rng(2).uniform(-1, 1, (1, 26)))
        P.semx_set_receivers(s.ctx, el, np.array([[1.0, 0.1, 0.2], [-1.0, 0.1, 0.2], [0.4, 0.5, 0.6], [1.0, 1.0, 1.0]]), 25)
        P.semx_set_dt(s.ctx, P.semx_cfl_dt(s.ctx, 0.3))
        P.semx_set_checkpointing(s.ctx, 7)
        P.semx_reset(s.ctx)
        P.semx_step(s.ctx, 25)
        g = torch.from_numpy(np.random.default_rng(4).standard_normal((1, 4, 3, 25)).astype(np.float32)).cuda()
        grads = [torch.empty((mesh.nspec, n ** 3), dtype=torch.float64, device="cuda") for _ in range(3)]
        P.semx_adjoint(s.ctx, g, 24, *grads)
        out.append([t.cpu().numpy() for t in grads])
        s.close()
    for a, b in zip(*out):
        # the terms of receivers at one node are added in another order: a rounding of 2^-24 a step, carried through
        # 24 steps of a recursion that preserves it
        assert np.linalg.norm(a - b) <= 24 * 6e-8 * 4 * np.linalg.norm(b)


@pytest.mark.parametrize("n,mode", [(2, "F32"), (5, "F32"), (10, "F32"), (12, "BF16"), (16, "F16"), (16, "F32"), (5, "BF16")])
@pytest.mark.parametrize("acoustic", [False, True])
@pytest.mark.parametrize("elements", [1, 3])
def test_nothing_to_sum(n, mode, acoustic, elements):
    """Elements that touch nowhere: an apply stores into f at once."""
    import paper_2606_12850_amd as P
    if acoustic and (mode != "F32" or n == 2):
        pytest.skip("no 16-bit contractions; the line kernel at NGLL 2")
    mesh = W.box_mesh((1, 1, 1), n, 1000.0)
    k = np.arange(elements)[:, None]
    mesh = SimpleNamespace(n=n, nspec=elements, nglob=elements * mesh.nglob,
                           ibool=(mesh.ibool + k * mesh.nglob).astype(np.int32),
                           elem_vert=(mesh.elem_vert + k * len(mesh.vert)).astype(np.int32),
                           vert=np.concatenate([mesh.vert + [2000.0 * e, 0.0, 0.0] for e in range(elements)]))
    kw = {"mode": None if mode == "F32" else getattr(P, "SEMX_C_" + mode), "acoustic": acoustic}
    for a, b in zip(_run(P, mesh, n, True, 0, **kw), _run(P, mesh, n, False, 0, **kw)):
        np.testing.assert_array_equal(a, b)
