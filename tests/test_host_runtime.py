"""The library's host code over a stub of the HIP runtime (no device): what
the calls that hand results back do when their launch is refused, what a
run's end waits for, how many launches a step takes."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"),
                                reason="needs g++ and the HIP headers")

# in a process of its own: the stub's symbols come before the HIP runtime's
PRELUDE = """
import ctypes as C, sys
import numpy as np
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
import paper_1507_03392_amd as ecr
import workloads as W
L = ecr.lib()

def create(n, **options):
    P, keep = ecr.make_params(W.with_(W.base_params(n, 8, 8, 16), **options))
    need = C.c_size_t()
    assert L.ecr_footprint(C.byref(P), C.byref(need)) == 0
    arena = np.zeros(need.value, dtype=np.uint8)
    run = C.c_void_p()
    assert L.ecr_create(C.byref(P), arena.ctypes.data, need.value, None, C.byref(run)) == 0
    assert L.ecr_init_ions(run) == 0
    return run, (arena, keep)

def view(n):
    a = {k: np.full(n, 7.0) for k in ("x", "y", "z", "vx", "vy", "vz")}
    a.update(q=np.full(n, 9, np.uint8), species=np.full(n, 9, np.uint8),
             cell=np.full(n, 9, np.uint32), birth=np.full(n, 9, np.uint32))
    return ecr.StateView(n=n, step=0, **{k: v.ctypes.data for k, v in a.items()}), a
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libstub.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I/opt/rocm/include", os.path.join(HERE, "hostcheck", "stub_hip.cpp"),
                    "-o", so], check=True, capture_output=True, text=True)
    return so


def host(stub, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, stub], capture_output=True, text=True, cwd=ROOT,
                       timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


@pytest.mark.parametrize("precision", [0, 1])
def test_a_refused_launch_is_an_error_of_the_read(stub, precision):
    host(stub, f"""
for at in (0, 1):  # the first read, and one after a good one
    run, keep = create(300, precision={precision})
    t = ecr.Tallies()
    for _ in range(at):
        assert L.ecr_read_tallies(run, C.byref(t)) == 0
    stub.stub_refuse(0)
    assert L.ecr_read_tallies(run, C.byref(t)) == -3
    assert b"read_tallies" in L.ecr_last_error(run)
for at in (0, 1):  # each of the launches of get_state
    run, keep = create(300, precision={precision})
    v, a = view(300)
    before = stub.stub_launches()
    assert L.ecr_get_state(run, C.byref(v)) == 0
    assert stub.stub_launches() == before + 2
    stub.stub_refuse(at)
    assert L.ecr_get_state(run, C.byref(v)) == -3
    assert b"get_state" in L.ecr_last_error(run)
run, keep = create(300, precision={precision})
v, a = view(300)
for k in ("q", "cell", "birth"):
    a[k][:] = 0
for at in range(3):
    stub.stub_refuse(at)
    assert L.ecr_set_state(run, C.byref(v)) == -3
    run, keep = create(300, precision={precision})
""")


def test_a_runs_end_waits_for_nothing(stub):
    # the tallies' pinned memory goes to the runs to come, a bounded part of
    # it; to free pinned memory waits for the whole device
    host(stub, """
t = ecr.Tallies()
for _ in range(100):  # one after another
    run, keep = create(40)
    assert L.ecr_read_tallies(run, C.byref(t)) == 0
    before = stub.stub_syncs(), stub.stub_host_frees()
    assert L.ecr_destroy(run) == 0
    assert (stub.stub_syncs(), stub.stub_host_frees()) == before
assert stub.stub_host_allocs() == 1
runs = [create(40) for _ in range(90)]  # at once
for r, _ in runs:
    assert L.ecr_read_tallies(r, C.byref(t)) == 0
assert stub.stub_host_allocs() == 90
for r, _ in runs:
    assert L.ecr_destroy(r) == 0
assert stub.stub_host_frees() == 90 - 64
# a run that failed may have a kernel about: its block is freed
run, keep = create(40)
assert L.ecr_read_tallies(run, C.byref(t)) == 0
stub.stub_refuse(0)
assert L.ecr_read_tallies(run, C.byref(t)) == -3
assert L.ecr_destroy(run) == 0
assert stub.stub_host_frees() == 90 - 64 + 1 and stub.stub_host_allocs() == 90
""")


def test_a_step_with_cell_grids_is_one_launch(stub):
    # and one for the exchange partners; a run of few particles on many cells
    # has two grids only, and a launch that clears the next one
    host(stub, """
for options, n, want in ((dict(self_ne=True), 3000, 1), (dict(self_n0=True), 3000, 1),
                         (dict(self_ne=True, self_n0=True, cx_partner=True), 3000, 2), (dict(self_ne=True), 100, 2),
                         (dict(), 3000, 1)):
    run, keep = create(n, process_mask=W.P_ALL | W.P_HEAT, **options)
    assert L.ecr_step(run, 1) == 0
    for _ in range(4):
        before = stub.stub_launches()
        assert L.ecr_step(run, 1) == 0
        assert stub.stub_launches() - before == want, (options, n)
""")
