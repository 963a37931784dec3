"""vof_read_planes around the number of cells (24576) up to which planes for
host arrays are split on the host instead of by a kernel: host and device
arrays, and any of the three alone, hold bitwise the same."""
from __future__ import annotations

import ctypes as C

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 29, 30])
def test_planes_on_both_routes(n):
    import torch

    import paper_1305_3417_amd as vof
    L = vof.lib()
    ctx = vof.vof_context_create(0)
    w = W.deform3d(n, steps=1)
    nc = w.mesh.n_cells
    print(f"[planes] {nc} cells", flush=True)
    m = vof.upload_mesh(ctx, w.mesh)
    vof.vof_set_alpha(m, w.alpha0)
    vof.vof_reconstruct(m)
    dev = [torch.zeros(k, dtype=t, device="cuda") for k, t in
           ((nc, torch.int8), (3 * nc, torch.float64), (nc, torch.float64))]
    assert L.vof_read_planes(m.h, *(C.c_void_p(d.data_ptr()) for d in dev), vof.VOF_DEVICE) == 0
    dev = [d.cpu().numpy() for d in dev]
    assert (dev[0] == 1).any() and np.isfinite(dev[2]).all()
    for want in ([0, 1, 2], [0], [1], [2], [1, 2]):
        host = [np.full_like(d, 7) for d in dev]
        args = [host[i].ctypes.data if i in want else None for i in range(3)]
        assert L.vof_read_planes(m.h, *args, vof.VOF_HOST) == 0
        for i in want:
            assert np.array_equal(host[i], dev[i])
    m.close()
    vof.vof_context_destroy(ctx)
