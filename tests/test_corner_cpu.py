"""The register clip's leading plane (one that keeps a single vertex of the
tetrahedron) where another vertex lies on that plane to rounding: the clip
finds the plane's side of each vertex in one place and the distances it cuts
with in another, so the corner has to be the same whichever side a rounding
puts that vertex on.  The closed-form self-test moves such a vertex onto the
plane and to either side, and returns NaN where the volume changes by more
than 1e-14 of the tetrahedron's.  Every vertex as the corner and as the vertex
on the plane; two to four planes."""
from __future__ import annotations

import itertools

import numpy as np
import pytest

import paper_1305_3417_amd as vof

# plane x <= 0: the first vertex is kept, the second is on the plane to
# rounding, the others are removed
TET = np.array([[-1.0, 0.25, 0.5], [0.0, 1.0, 0.25], [1.0, 0.125, -0.5], [0.75, 0.0, 1.0]])
OTHERS = np.array([[0.5, 1.0, 0.25, 0.5], [-0.25, 0.5, 1.0, 0.625], [0.125, -1.0, 0.5, 0.25]])


@pytest.mark.parametrize("off", [1e-18, 2e-16, 4e-16])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_vertex_on_the_leading_plane(k, off):
    T0 = TET.copy()
    T0[1, 0] = off
    planes = np.concatenate([[[1.0, 0.0, 0.0, 0.0]], OTHERS[:k]])
    cut = vof.vof_selftest_tet_clip(T0, planes)
    whole = abs(np.linalg.det(T0[1:] - T0[0])) / 6
    assert 0.01 * whole < cut < 0.5 * whole
    for order in itertools.permutations(range(4)):
        a = vof.vof_selftest_tet_clip_closed(T0[list(order)], planes)
        assert abs(a - cut) <= 1e-15, (order, a, cut)
