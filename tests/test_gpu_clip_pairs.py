"""The register clip's count of overlapping (flux tet, cell) pairs on box cells
of a refined mesh, against a count in NumPy with the same vertices: points less
the rounded face centre, as the cells' planes are taken against that centre.  A
point on a cell's side then has the distance 0 and cuts nothing; with the
subtraction fused into the centre's last product it lies a rounding off the
side wherever the mean over three, five or more points is rounded, and the clip
evaluates pairs that only touch (1 % more on these meshes).

Every cell holds 0.37, so every face with flux is clipped; the velocity is
uniform and oblique, so no tet is flat and only face points meet sides."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from workloads import fields
from workloads.refine import refine_hex

pytestmark = pytest.mark.gpu


def _workload(n):
    k, j, i = (x.ravel() for x in np.meshgrid(*[np.arange(n)] * 3, indexing="ij"))
    mesh, _, _ = refine_hex(n, (i % 3 == 1) & (j % 3 == 1) & (k % 3 == 1))
    U = np.array([0.3, -0.2, 0.1])
    return W.Workload("oblique", mesh, np.full(mesh.n_cells, 0.37),
                      np.tile(U, (mesh.n_cells, 1)), fields.flux_constant(mesh, U),
                      np.array([0.25 / n]), np.ones(1))


def _pair_count(w, lam, Up):
    m = w.mesh
    lo, hi = np.full((m.n_cells, 3), np.inf), np.full((m.n_cells, 3), -np.inf)
    cells_of = [set() for _ in range(m.n_points)]
    for f in range(m.n_faces):
        p = m.face_points[m.face_offsets[f]:m.face_offsets[f + 1]]
        for c in [m.owner[f]] + ([m.neighbour[f]] if f < m.n_internal else []):
            lo[c] = np.minimum(lo[c], m.points[p].min(0))
            hi[c] = np.maximum(hi[c], m.points[p].max(0))
            for q in p:
                cells_of[q].add(int(c))
    count = 0
    for f in np.flatnonzero(w.F0 != 0.0):
        p = m.face_points[m.face_offsets[f]:m.face_offsets[f + 1]]
        n = len(p)
        x = np.zeros((8, 3))
        x[:n] = m.points[p]
        u = np.zeros((8, 3))
        u[:n] = (-w.scale[0] * w.dt[0] * lam[f]) * Up[p]
        s, su = x, u  # sums over pairs of lanes, as the kernel adds them
        while len(s) > 1:
            s, su = s[::2] + s[1::2], su[::2] + su[1::2]
        c = (1.0 / n) * s[0]
        top = (1.0 / n) * su[0]
        P = x[:n] - c
        Q = P + u[:n]
        Pn, Qn = np.roll(P, -1, 0), np.roll(Q, -1, 0)
        M = 0.25 * (P + Pn + Q + Qn)
        T = np.broadcast_to(top, P.shape)
        tets = np.stack([np.stack(t) for t in
                         ((T, Qn, Q), (M, Pn, P), (M, P, Q), (M, Q, Qn), (M, Qn, Pn))])
        tets = tets.transpose(0, 2, 1, 3).reshape(-1, 3, 3)   # tet, vertex, axis
        verts = np.concatenate([np.zeros((len(tets), 1, 3)), tets], 1)
        # cells that meet the polyhedron's box (not only touch it)
        cells = np.array(sorted(set().union(*(cells_of[q] for q in p))))
        ends = np.concatenate([x[:n], x[:n] + u[:n]])
        cells = cells[((ends.max(0) > lo[cells]) & (ends.min(0) < hi[cells])).all(1)]
        up = (hi[cells] - c)[None, :, None, :] - verts[:, None]
        dn = (c - lo[cells])[None, :, None, :] + verts[:, None]
        hit = ((up > 0).any(2) & (dn > 0).any(2)).all(2)       # tet, cell
        inside = hit & ~((up < 0) | (dn < 0)).any((2, 3))
        before = np.cumsum(inside, 1) - inside == 0            # up to the first it lies in
        count += int((hit & before).sum())
    return count


@pytest.mark.parametrize("n", [6, 9])
def test_touching_cells_are_no_pairs(n):
    import paper_1305_3417_amd as vof
    w = _workload(n)
    ctx = vof.vof_context_create(0)
    m = vof.upload_mesh(ctx, w.mesh)
    vof.vof_set_alpha(m, w.alpha0)
    vof.vof_set_velocity(m, w.U0c, w.F0)
    vof.vof_advect(m, w.dt, w.scale)
    s = vof.vof_get_stats(m)
    want = _pair_count(w, vof.vof_read_face(m, vof.VOF_FACE_LAMBDA),
                       vof.vof_read_point_velocity(m).reshape(-1, 3))
    print(f"[pairs] {w.mesh.n_cells} cells: {s['clip_pairs']} pairs, {want} counted", flush=True)
    assert s["general_tets"] == 0 and s["unreached_faces"] == 0
    assert s["geometric_faces"] == (w.F0 != 0.0).sum()
    assert s["clip_pairs"] == want
    m.close()
    vof.vof_context_destroy(ctx)
