"""The device's closed-form kept fraction (whose quotient is no IEEE division)
over length units from 1e-36 to 1e30: mapping a reconstructed field to the
eight children of every cell evaluates it on other tetrahedra than the
positioning did, so the children of an interface cell hold the cell's phase
volume again only if both are right to rounding.

Bound: an evaluation adds 24 fan tetrahedra of a box, each fraction good to a
few eps (eps = 2.2e-16) of its volume, together 16 eps of the box at the most;
so does the positioning, which also stops at 1e-15.  2 * 16 eps + 1e-15 < 1e-14."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from workloads.refine import refine_hex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exponent", [-120, 0, 100])
def test_children_hold_their_cells_volume(exponent):
    import paper_1305_3417_amd as vof
    n = 12
    w = W.deform3d(n, steps=1)
    fine, _, (_, kids) = refine_hex(n, np.ones(n ** 3, dtype=bool))
    parent = np.repeat(np.arange(n ** 3), 8)
    alpha = np.random.default_rng(7).uniform(1e-3, 1.0 - 1e-3, n ** 3)
    ctx = vof.vof_context_create(0)
    src, dst = (vof.vof_mesh_upload(ctx, np.ldexp(m.points, exponent), m.face_offsets,
                                    m.face_points, m.owner, m.neighbour, m.n_cells)
                for m in (w.mesh, fine))
    vof.vof_set_alpha(src, alpha)
    order = np.empty(fine.n_cells, dtype=np.int32)
    order[kids] = parent  # the cell each fine cell lies in
    print(f"[kept fraction] length unit 2^{exponent}", flush=True)
    vof.vof_map_alpha(dst, src, np.arange(fine.n_cells + 1, dtype=np.int32), order)
    cls, _, _ = vof.vof_read_planes(src)
    got = vof.vof_read_alpha(dst)[kids].reshape(-1, 8)
    assert (cls == 1).sum() > 1000
    assert np.ptp(got, axis=1).max() > 0.9
    assert np.abs(got.mean(axis=1) - alpha)[cls == 1].max() < 1e-14
    src.close()
    dst.close()
    vof.vof_context_destroy(ctx)
