"""Mass, range and counters of vof_get_stats (two reduction stages) on meshes
of less than a block to more blocks than the first stage has.

The mass is a compensated sum of V alpha: on cubes of volume h^3 (known to a
few roundings of the geometry kernel) it meets the exact sum to 1e-14
relative; minimum and maximum are exact."""
from __future__ import annotations

import math

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 13, 41, 129])
def test_mass_and_range(n):
    import paper_1305_3417_amd as vof
    w = W.deform3d(n, steps=1)
    ctx = vof.vof_context_create(0)
    m = vof.upload_mesh(ctx, w.mesh)
    alpha = np.random.default_rng(n).uniform(-1e-3, 1.0, w.mesh.n_cells)
    print(f"[stats] {alpha.size} cells", flush=True)
    vof.vof_set_alpha(m, alpha)
    s = vof.vof_get_stats(m)
    exact = math.fsum(alpha) / n**3
    assert abs(s["mass"] - exact) <= 1e-14 * abs(exact)
    assert s["alpha_min"] == alpha.min() and s["alpha_max"] == alpha.max()
    assert s["steps"] == 0 and s["geometric_faces"] == 0 and s["ledger"] == 0.0
    m.close()
    vof.vof_context_destroy(ctx)
