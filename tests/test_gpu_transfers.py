"""What goes in and out of a mesh beside the steps: a velocity field set again
before a call and a call of few steps after one of many (whose schedule array
stays) give bitwise the run of single steps, and the planes read are those of
the reconstruction (unit normals in interface cells, zero where no plane was
ever set).  Cell counts below, at and above a block."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _mesh(vof, ctx, w, device):
    import torch
    m = vof.upload_mesh(ctx, w.mesh)
    vof.vof_set_alpha(m, torch.from_numpy(w.alpha0).cuda() if device else w.alpha0)
    vof.vof_set_velocity(m, w.U0c, w.F0)
    return m


@pytest.mark.parametrize("n", [6, 16, 21])
def test_velocities_schedules_and_planes(n):
    import paper_1305_3417_amd as vof
    ctx = vof.vof_context_create(0)
    w = W.deform3d(n, steps=700)
    print(f"[transfers] {w.mesh.n_cells} cells", flush=True)
    out = []
    for device, calls in ((False, [3, 2]), (True, [3, 2]), (False, [1] * 5)):
        m = _mesh(vof, ctx, w, device)
        if calls[0] == 3:  # a schedule array of 600 entries first, then back to the start
            vof.vof_advect(m, w.dt[:600], w.scale[:600])
            vof.vof_set_alpha(m, w.alpha0)
        at = 0
        for k in calls:
            vof.vof_set_velocity(m, w.U0c, w.F0)
            vof.vof_advect(m, w.dt[at:at + k], w.scale[at:at + k])
            at += k
        cls, normal, s = vof.vof_read_planes(m)
        out.append((vof.vof_read_alpha(m), vof.vof_read_face(m, vof.VOF_FACE_VPHASE), cls, normal, s))
        length = np.linalg.norm(normal, axis=1)
        assert np.abs(length[cls == 1] - 1.0).max() < 1e-14
        assert np.isfinite(s).all() and (np.abs(s[length == 0.0]) == 0.0).all()
        m.close()
    for o in out[1:]:
        for a, b in zip(o, out[0]):
            assert np.array_equal(a, b)
    vof.vof_context_destroy(ctx)
