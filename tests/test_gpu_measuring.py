"""What the timing calls count and compare: launches of a pass, and the memory
skeleton of the kernel that runs.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _solver(n, ne, jitter=0.1):
    import paper_2606_12850_amd as P
    mesh = W.box_mesh(ne, n, 4000.0, jitter=jitter, seed=3)
    s = P.Solver(n)
    s.upload_mesh(mesh)
    P.semx_set_geometry(s.ctx, P.SEMX_GEOM_TRILINEAR)
    s.upload_model(*W.homogeneous_model(mesh))
    return P, s, mesh


def test_launches_counted():
    """Element-local forces: one launch for the mesh's kind of element, and in an apply the nodal sum."""
    import torch
    P, s, mesh = _solver(5, 6)
    u = torch.rand((mesh.nglob, 3), device="cuda")
    f = torch.empty_like(u)
    P.semx_set_timing(s.ctx, 1)
    for _ in range(3):
        P.semx_apply_force(s.ctx, u, f)
    n, ms = P.semx_force_timing(s.ctx)
    assert n == 3 * 2 and ms > 0
    P.semx_set_dt(s.ctx, P.semx_cfl_dt(s.ctx, 0.3))
    s.step(4)
    n, ms = P.semx_force_timing(s.ctx)
    assert n == 4 and ms > 0
    s.set_mode(P.SEMX_C_F32, P.SEMX_ASM_ATOMIC)
    P.semx_apply_force(s.ctx, u, f)
    n, ms = P.semx_force_timing(s.ctx)
    assert n == 1 and ms > 0
    s.close()


@pytest.mark.parametrize("n,ne,jitter", [(2, 90, 0.1), (5, 40, 0.1), (8, 22, 0.0), (10, 16, 0.1), (12, 11, 0.0)])
def test_skeleton_of_the_line_kernel(n, ne, jitter):
    """The pass takes no less time than its memory skeleton (within the spread of two timings) and is left unchanged."""
    import torch
    P, s, mesh = _solver(n, ne, jitter)
    u = torch.rand((mesh.nglob, 3), device="cuda")
    f = torch.empty_like(u)
    P.semx_apply_force(s.ctx, u, f)
    want = f.clone()
    sk = min(P.semx_force_skeleton(s.ctx, u, f, 20) for _ in range(3))
    P.semx_set_timing(s.ctx, 1)
    for _ in range(20):
        P.semx_apply_force(s.ctx, u, f)
    _, ms = P.semx_force_timing(s.ctx)
    torch.cuda.synchronize()
    print(f"n={n}: skeleton {sk * 1e3:.1f} us, pass {ms / 20 * 1e3:.1f} us")
    assert 0.0 < sk <= 1.1 * ms / 20
    assert torch.equal(f, want)
    s.close()
