"""The register clip's face groups and claims.

A face's phase volume does not depend on the group it is clipped in: a small
hexahedral mesh alone takes groups of one tet per lane, in a batch beside a
mesh with many geometric faces groups of two, with other chunk and round
boundaries, and its alpha and V_alpha are bitwise the same.  Nor on the claims:
grids below and off the eight XCDs, and claims of one and of several groups,
visit every group once.  Faces of three, four and up to eight points (the
tets per lane go by the faces of a mesh's own kind, so the refined and the
tetrahedral mesh keep one here and vary the claims only)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SMALL = {"hex": lambda k: W.deform3d(10, steps=k), "refined": lambda k: W.deform3d_refined(8, steps=k),
         "tets": lambda k: W.rotate_tets(5, steps=k, sample=4)}


@pytest.fixture(scope="module")
def vof():
    import torch
    assert torch.cuda.is_available()
    import paper_1305_3417_amd as vof
    vof.lib()
    return vof


@pytest.fixture(scope="module")
def large():
    return W.deform3d(60, steps=2)


def _upload(vof, ctx, w):
    m = vof.upload_mesh(ctx, w.mesh)
    vof.vof_set_alpha(m, w.alpha0)
    vof.vof_set_velocity(m, w.U0c, w.F0)
    return m


def _state(vof, m):
    return vof.vof_read_alpha(m), vof.vof_read_face(m, vof.VOF_FACE_VPHASE)


@pytest.mark.parametrize("grid,claim", [(4096, 2), (5, 3), (13, 1)])
@pytest.mark.parametrize("kind", sorted(SMALL))
def test_groups_and_claims_do_not_change_results(vof, large, kind, grid, claim):
    ctx = vof.vof_context_create(0)
    ws = [SMALL[kind](2), large]
    alone = []
    for w in ws:
        m = _upload(vof, ctx, w)
        vof.vof_advect(m, w.dt[:2], w.scale[:2])
        alone.append(_state(vof, m))
        faces = vof.vof_get_stats(m)["geometric_faces"] / 2
        print(f"[{kind}] {w.mesh.n_cells} cells, {faces} geometric faces a step", flush=True)
        m.close()
    # the large mesh takes two tets per lane, the small one alone does not
    assert faces > 2048 * 3
    meshes = [_upload(vof, ctx, w) for w in ws]
    b = vof.vof_batch_create(ctx, meshes)
    c = vof.vof_batch_get_config(b)
    c.grid_clip, c.clip_claim = grid, claim
    vof.vof_batch_set_config(b, c)
    vof.vof_batch_advect(b, np.stack([w.dt[:2] for w in ws]), np.stack([w.scale[:2] for w in ws]))
    vof.vof_batch_synchronize(b)
    for m, (alpha, vphase) in zip(meshes, alone):
        a, v = _state(vof, m)
        assert np.array_equal(a, alpha) and np.array_equal(v, vphase)
    vof.vof_batch_destroy(b)
    for m in meshes:
        m.close()
    vof.vof_context_destroy(ctx)
