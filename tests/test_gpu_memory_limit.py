"""What fits without the element-local forces fits: they make room.

The element-local forces of a pass are optional (without them the pass runs
colour by colour, with the same sums).  On a device whose memory is counted and
limited (tests/native/limited_memory.cpp) a model is accepted with no more
memory than its upload takes under a colouring of the caller's, which has no
element-local forces, and records, checkpoints and the adjoint's buffers that
leave no room for them are accepted too, with unchanged results.  The points of
a node of a structured box follow from its place: no tables are kept.
"""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))

SCRIPT = r"""
import ctypes, sys
M = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
for name in ("limited_used", "limited_peak"):
    getattr(M, name).restype = ctypes.c_uint64
M.limited_set.argtypes = [ctypes.c_uint64]
import numpy as np
import torch
import paper_2606_12850_amd as P
import workloads as W

n, ne, kind = 5, 6, sys.argv[2]
mesh = W.box_mesh(ne, n, 4000.0, jitter=0.1, seed=2)
model = W.layered_model(mesh)
f64 = kind == "upload64"
part = (24 if f64 else 12) * mesh.nspec * n ** 3
gen = torch.Generator("cuda").manual_seed(1)


def solver(own_colours=False, limit=0):
    s = P.Solver(n, storage=P.SEMX_F64 if f64 else P.SEMX_F32)
    P.semx_set_geometry(s.ctx, P.SEMX_GEOM_TRILINEAR)  # no element blocks
    s.upload_mesh(mesh)
    if own_colours:
        P.semx_set_coloring(s.ctx, *P.semx_get_coloring(s.ctx, mesh.nspec))
    base = M.limited_used()
    M.limited_set(base + limit if limit else 0)
    s.upload_model(*model)
    s.peak = M.limited_peak() - base
    M.limited_set(0)
    return s


def forces(s, u):
    f = s.apply_force(u)
    torch.cuda.synchronize()
    return f.cpu().numpy()


ref = solver()
u = ref.empty_field().normal_(generator=gen)
want = forces(ref, u)
assert M.limited_used() > part, "allocations are not counted"
if kind == "tables":
    used = []
    for scrambled in (False, True):
        m = W.box_mesh(ne, n, 4000.0)
        if scrambled:
            m.ibool = np.random.default_rng(1).permutation(m.nglob).astype(np.int32)[m.ibool]
        s = P.Solver(n)
        base = M.limited_used()
        s.upload_mesh(m)
        used.append(M.limited_used() - base)
        s.upload_model(*W.homogeneous_model(m))
        s.close()
    assert used[1] - used[0] >= 4 * mesh.nspec * n ** 3, used  # a lattice keeps no node tables
elif kind.startswith("upload"):
    own = solver(own_colours=True)
    s = solver(limit=own.peak)
    np.testing.assert_array_equal(forces(s, u), want)
    np.testing.assert_array_equal(forces(own, u), want)
else:
    nt, every = 12, 4
    def run(s, limit):
        P.semx_set_sources(s.ctx, *W.center_vertex_source(mesh), np.array([[0.3, -0.2, 1.0]]),
                           1e9 * np.sin(np.arange(nt + 1, dtype=np.float32))[None, :])
        P.semx_set_dt(s.ctx, P.semx_cfl_dt(s.ctx, 0.3))
        rec, xi = np.zeros(8, np.int32), np.zeros((8, 3))
        P.semx_set_receivers(s.ctx, rec, xi, nt)
        base = M.limited_used()
        if kind == "records":
            more = 10 * part                                       # bytes of longer records
            M.limited_set(base + more - part // 2 if limit else 0)
            P.semx_set_receivers(s.ctx, rec, xi, more // (8 * 3 * 4))
            M.limited_set(0)
            P.semx_set_receivers(s.ctx, rec, xi, nt)
            P.semx_reset(s.ctx)
            s.step(nt)
        else:
            P.semx_set_checkpointing(s.ctx, every)
            four = 4 * 36 * mesh.nglob                             # bytes of the run's four checkpoints
            M.limited_set(base + four - part // 2 if limit and kind == "checkpoints" else 0)
            P.semx_reset(s.ctx)
            s.step(nt)
            base = M.limited_used()
            work = 24 * mesh.nspec * n ** 3 + 18 * 12 * mesh.nglob  # bytes of the adjoint's buffers
            M.limited_set(base + work - part // 2 if limit and kind == "adjoint" else 0)
            g = [torch.empty((mesh.nspec, n ** 3), dtype=torch.float64, device="cuda") for _ in range(3)]
            w = torch.randn((1, 8, 3, nt), device="cuda", generator=torch.Generator("cuda").manual_seed(2))
            P.semx_adjoint(s.ctx, w, nt, *g)
            s.grads = [x.cpu().numpy() for x in g]
            M.limited_set(0)
        a, v = s.empty_field(), s.empty_field()
        P.semx_get_state(s.ctx, a, v)
        torch.cuda.synchronize()
        s.out = [a.cpu().numpy(), v.cpu().numpy()]
    s = solver()
    run(ref, False)
    run(s, True)
    for x, y in zip(ref.out, s.out):
        assert np.abs(x).max() > 0
        np.testing.assert_array_equal(x, y)
    for x, y in zip(getattr(ref, "grads", []), getattr(s, "grads", [])):
        # receivers that share a node add in FP64 with element-local forces, in FP32 without
        assert np.linalg.norm(x - y) <= 1e-5 * np.linalg.norm(x)
    np.testing.assert_array_equal(forces(s, u), want)
    s.close()
print("ok")
"""


@pytest.fixture(scope="module")
def limited(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("native") / "limited_memory.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", os.path.join(HERE, "native", "limited_memory.cpp"), "-o", so, "-ldl"],
                   check=True)
    return so


@pytest.mark.parametrize("kind", ["upload", "upload64", "records", "checkpoints", "adjoint", "tables"])
def test_room_is_made(limited, kind):
    r = subprocess.run([sys.executable, "-c", SCRIPT, limited, kind], cwd=os.path.dirname(HERE), capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.stdout + r.stderr)[-2000:]
