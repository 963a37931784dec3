"""The register clip with two flux tets per lane on faces of more than four
points: meshes whose largest faces have five, six and eight points, with more
geometric faces than one-tet-per-lane groups fill the chip with (6144), so
that a group holds up to five large faces (five of five points fill the
vertex rows to the last), its tets span both ballot words, and a face's tets
take two batches.

Every cell is an interface cell (random alpha), so every face with flux is
clipped.  One step against the oracle (V_alpha to the tolerance of the parity
tests: 1e-12 of the face's swept volume or of a hundredth of its cell), and a
small mesh of the same kind, alone in groups of one tet per lane, bitwise the
same beside the large one in groups of two."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from tests.common import gpu_run, oracle_run, vphase_tolerance
from workloads import fields
from workloads.refine import refine_hex

pytestmark = pytest.mark.gpu

# refined cells by their indices; the points of the largest face
PATTERNS = {5: lambda i, j, k: (i % 3 == 1) & (j % 3 == 1) & (k % 3 == 1),
            6: lambda i, j, k: ((i + j) % 3 == 0) & (k % 3 == 1),
            8: lambda i, j, k: (i + j + k) % 3 == 0}


def _workload(points, n, steps):
    k, j, i = (x.ravel() for x in np.meshgrid(*[np.arange(n)] * 3, indexing="ij"))
    mesh, _, _ = refine_hex(n, PATTERNS[points](i, j, k))
    assert np.diff(mesh.face_offsets).max() == points
    alpha = np.random.default_rng(points + n).uniform(0.02, 0.98, mesh.n_cells)
    return W.Workload(f"refined{points}", mesh, alpha,
                      fields.deformation_velocity(mesh.cell_centroids()),
                      fields.flux_deformation(mesh), np.full(steps, 1.0 / (8 * n)), np.ones(steps))


@pytest.fixture(scope="module")
def vof():
    import torch
    assert torch.cuda.is_available()
    import paper_1305_3417_amd as vof
    vof.lib()
    return vof


@pytest.mark.parametrize("points", sorted(PATTERNS))
def test_two_tets_per_lane(vof, oracle_mod, points):
    ctx = vof.vof_context_create(0)
    small, large = _workload(points, 6, 1), _workload(points, 18, 1)
    alone = []
    for w in (small, large):
        g = gpu_run(vof, ctx, w)
        faces = g["stats"]["geometric_faces"]
        print(f"[{points} points] {w.mesh.n_cells} cells, {faces} geometric faces", flush=True)
        assert (faces > 6144) == (w is large) and faces > 500
        o, a, _, _, vp = oracle_run(oracle_mod, w)
        V, _, S, _ = o.geometry()
        Up = o.set_velocity(w.U0c, w.F0)
        tol = vphase_tolerance(w, V, w.dt[0], S, Up)
        assert (np.abs(g["vphase"] - vp) <= tol).all()
        alone.append((g["alpha"], g["vphase"]))
        g["mesh"].close()
    ws = (small, large)
    meshes = [vof.upload_mesh(ctx, w.mesh) for w in ws]
    for m, w in zip(meshes, ws):
        vof.vof_set_alpha(m, w.alpha0)
        vof.vof_set_velocity(m, w.U0c, w.F0)
    b = vof.vof_batch_create(ctx, meshes)
    vof.vof_batch_advect(b, np.stack([w.dt for w in ws]), np.stack([w.scale for w in ws]))
    vof.vof_batch_synchronize(b)
    for m, (alpha, vphase) in zip(meshes, alone):
        assert np.array_equal(vof.vof_read_alpha(m), alpha)
        assert np.array_equal(vof.vof_read_face(m, vof.VOF_FACE_VPHASE), vphase)
    vof.vof_batch_destroy(b)
    for m in meshes:
        m.close()
    vof.vof_context_destroy(ctx)
