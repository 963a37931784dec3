"""Range and mass of vof_get_stats where alpha holds values that are no
numbers: a field of nothing but NaN has no range, one with some of them the
range of the other cells, and the mass is NaN in both.  Meshes of less than a
block, and of more cells than the first reduction stage takes in one pass."""
from __future__ import annotations

import math

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 41, 82])
def test_range_of_nan(n):
    import paper_1305_3417_amd as vof
    w = W.deform3d(n, steps=1)
    ctx = vof.vof_context_create(0)
    m = vof.upload_mesh(ctx, w.mesh)
    nc = w.mesh.n_cells
    print(f"[stats] {nc} cells", flush=True)
    vof.vof_set_alpha(m, np.full(nc, np.nan))
    s = vof.vof_get_stats(m)
    assert math.isnan(s["alpha_min"]) and math.isnan(s["alpha_max"]) and math.isnan(s["mass"])
    alpha = np.random.default_rng(n).uniform(-1e-3, 1.0, nc)
    alpha[::3] = np.nan
    alpha[-1] = np.nan
    vof.vof_set_alpha(m, alpha)
    s = vof.vof_get_stats(m)
    assert s["alpha_min"] == np.nanmin(alpha) and s["alpha_max"] == np.nanmax(alpha)
    assert math.isnan(s["mass"])
    m.close()
    vof.vof_context_destroy(ctx)
