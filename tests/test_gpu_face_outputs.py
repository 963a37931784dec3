"""Per-face outputs after calls of several steps: the last step of a call
writes every face's lambda, iterations, kind and status, whatever the steps
before it left, so one call of three steps reads bitwise as calls of two and
one; likewise the phase volumes and alpha (a cell without phase flux is
skipped by the update).  The interface moves, so faces change kind."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = {"hex": lambda: W.deform3d(20, steps=9), "tets": lambda: W.rotate_tets(6, steps=9, sample=4),
         "refined": lambda: W.deform3d_refined(8, steps=9), "disc": lambda: W.disc2d(24, steps=9)}


def _run(vof, w, calls, batch, **params):
    ctx = vof.vof_context_create(0)
    m = vof.upload_mesh(ctx, w.mesh)
    if params:
        p = vof.vof_get_params(m)
        for k, v in params.items():
            setattr(p, k, v)
        vof.vof_set_params(m, p)
    vof.vof_set_alpha(m, w.alpha0)
    vof.vof_set_velocity(m, w.U0c, w.F0)
    b = vof.vof_batch_create(ctx, [m]) if batch else None
    at = 0
    for k in calls:
        if batch:
            vof.vof_batch_advect(b, w.dt[None, at:at + k], w.scale[None, at:at + k])
            vof.vof_batch_synchronize(b)
        else:
            vof.vof_advect(m, w.dt[at:at + k], w.scale[at:at + k])
        at += k
    out = [vof.vof_read_alpha(m)] + [vof.vof_read_face(m, what) for what in (
        vof.VOF_FACE_LAMBDA, vof.VOF_FACE_VPHASE, vof.VOF_FACE_ITERS, vof.VOF_FACE_KIND,
        vof.VOF_FACE_STATUS)]
    if b:
        vof.vof_batch_destroy(b)
    m.close()
    vof.vof_context_destroy(ctx)
    return out


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("band", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_last_step_writes_every_face(case, band, batch):
    import paper_1305_3417_amd as vof
    w = CASES[case]()
    print(f"[{case}] band {band} batch {batch}", flush=True)
    every = _run(vof, w, [1] * 9, batch, narrow_band=band)
    for calls in ([9], [5, 1, 3]):
        for a, b in zip(_run(vof, w, calls, batch, narrow_band=band), every):
            assert np.array_equal(a, b)
    assert len(np.unique(every[4])) > 2  # several kinds of faces
