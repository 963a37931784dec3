"""The library's host code without a GPU, on a stand-in for the HIP runtime
(fake_hip.cpp: device memory is host memory, kernels are noted and not run):
what a call copies, launches and waits for, and what it does where a copy or a
host allocation fails.  Each test runs in a process of its own, with the
stand-in loaded before the library."""
from __future__ import annotations

import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, sys
import numpy as np
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.fake_fail_new.argtypes = [C.c_size_t]
fake.fake_fail_copy.argtypes = [C.c_long]
fake.fake_log_stop.restype = C.c_char_p
import paper_1305_3417_amd as vof
import workloads as W

def logged(fn):
    fake.fake_log_start()
    try:
        fn()
    finally:
        lines = fake.fake_log_stop().decode().splitlines()
    out = []
    for ln in lines:
        what, a, b = ln.rsplit(" ", 2)
        out.append((what, int(a), int(b)))
    return out

def upload(w):
    m = vof.upload_mesh(ctx, w.mesh)
    vof.vof_set_alpha(m, w.alpha0)
    vof.vof_set_velocity(m, w.U0c, w.F0)
    return m

ctx = vof.vof_context_create(0, stream=0)
"""


@pytest.fixture(scope="module")
def fake_hip(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-o", so,
                           os.path.join(HERE, "fake_hip.cpp")])
    return so


def run(fake_hip, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), fake_hip],
                       cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


def test_schedules_need_no_host_memory(fake_hip):
    """vof_advect stages the schedule without a host allocation of its size:
    calls of one to many steps, before and after longer ones, pass where every
    allocation of 1 KiB or more fails, and copy dt and scale."""
    run(fake_hip, """
    w = W.deform3d(4, steps=5000)
    m = upload(w)
    fake.fake_fail_new(1024)
    for n in (1, 200, 2, 511, 512, 513, 3, 1100, 700, 5000, 1):
        got = logged(lambda: vof.vof_advect(m, w.dt[:n], w.scale[:n]))
        assert sum(g[0] == "graph" for g in got) == n
        assert sum(g[2] for g in got if g[0] == "to_device") >= 16 * n
    """)


@pytest.mark.parametrize("memory", ["host", "device"])
def test_failed_velocity_is_not_used(fake_hip, memory):
    """Where a copy of vof_set_velocity fails, no later step runs on a mixture
    of two fields: either nothing was launched, so that the earlier velocity
    still stands, or the mesh has no velocity.  Of device arrays the earlier
    velocity always stands."""
    run(fake_hip, f"\n    memory = {int(memory == 'device')}" + """
    w = W.deform3d(4, steps=1)
    def set_velocity(m):
        U, F = 2.0 * w.U0c, 2.0 * w.F0
        return vof.lib().vof_set_velocity(m.h, U.ctypes.data, F.ctypes.data, memory)
    def kernels(got):
        return [g for g in got if g[0].startswith("kernel")]
    def stands(m):
        return vof.lib().vof_advect(m.h, 1, w.dt.ctypes.data, w.scale.ctypes.data) == vof.VOF_OK
    for nth in (1, 2):
        m = upload(w)
        assert len(kernels(logged(lambda: set_velocity(m)))) > 0 and stands(m)
        fake.fake_fail_copy(nth)
        codes = []
        got = kernels(logged(lambda: codes.append(set_velocity(m))))
        assert codes == [vof.VOF_EDEVICE]
        assert stands(m) == (got == []), nth
        assert got == [] or not memory
        assert set_velocity(m) == vof.VOF_OK and stands(m)
    """)


def test_planes_of_small_meshes_in_one_copy(fake_hip):
    """vof_read_planes of a mesh of up to 24576 cells for host arrays: one copy
    of the classes, one of the planes and no kernel, whichever arrays are
    asked for; of more cells a kernel splits the planes first."""
    run(fake_hip, """
    for n, kernels, copies in ((4, 0, 2), (28, 0, 2), (30, 1, 3)):
        w = W.deform3d(n, steps=1)
        m = vof.upload_mesh(ctx, w.mesh)
        vof.vof_set_alpha(m, w.alpha0)
        got = logged(lambda: vof.vof_read_planes(m))
        assert sum(g[0].startswith("kernel") for g in got) == kernels, n
        assert sum(g[0] == "to_host" for g in got) == copies, n
        s = np.empty(w.mesh.n_cells)
        fake.fake_fail_new(1024)  # also where the host has no room for a copy
        assert vof.lib().vof_read_planes(m.h, None, None, s.ctypes.data, 0) == vof.VOF_OK
        fake.fake_fail_new(0)
    """)


def test_autotuner_times_the_step_that_runs(fake_hip):
    """The autotuner's timed steps launch the clips of two and three face kinds
    side by side as the captured step does: the same kernels on the same
    number of streams, between the same fork and join."""
    run(fake_hip, """
    kinds = {"tets": W.rotate_tets(3, steps=4, sample=2), "hex": W.deform3d(4, steps=4),
             "refined": W.deform3d_refined(4, steps=4)}
    for names in (["hex"], ["tets", "hex"], ["hex", "refined"], ["tets", "hex", "refined"]):
        ms = [upload(kinds[k]) for k in names]
        b = vof.vof_batch_create(ctx, ms)
        dt = np.stack([kinds[k].dt[:4] for k in names])
        sc = np.stack([kinds[k].scale[:4] for k in names])
        clips = {}
        for what, fn in (("timed", vof.vof_autotune), ("run", vof.vof_batch_advect)):
            got = logged(lambda: fn(b, dt, sc))
            c = [g for g in got if "kb_clip_fast" in g[0]]
            if what == "timed":
                assert len(c) == 4 * len(names)
                c = c[:len(names)]
            main = next(g[1] for g in got if "kb_group_prefix" in g[0])
            clips[what] = [(g[0], g[1] != main) for g in c]
        assert clips["timed"] == clips["run"], names
        assert sum(aside for _, aside in clips["run"]) == (len(names) > 1)
        vof.vof_batch_destroy(b)
    """)
