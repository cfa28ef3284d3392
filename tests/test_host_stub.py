"""Host logic of a solve without a GPU: the library on a stand-in HIP runtime (hip_stub.hip), whose
kernels do nothing and whose failures the tests choose.  In a child process, which loads the
stand-in before the library."""
import os
import subprocess
import sys

import pytest

import paper_2607_26082_amd.build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C, sys
sys.path.insert(0, {root!r})
stub = C.CDLL({stub!r}, mode=C.RTLD_GLOBAL)
stub.stub_word.restype = C.c_void_p
sys.modules["torch"] = None              # no second runtime in this process
import numpy as np
import paper_2607_26082_amd as F
lib = F.load()
buf = np.zeros((64 << 20) + 256, np.uint8)
WS = (buf.ctypes.data + 255) // 256 * 256
LAM = np.ones(16 ** 3); MU = np.ones(16 ** 3)

def handle(n=(16, 16, 16), prec=F.FFTC_FP64, bc=None, bytes=64 << 20):
    h = F.fftc_create(n, prec)
    if bc is not None:
        F.fftc_set_bc(h, bc)
    F.fftc_set_reference(h, 1.0, 1.0)
    F.fftc_set_solver(h, tol=0.0, max_iter=50)
    rc = lib.fftc_bind_workspace(h, C.c_void_p(WS), C.c_size_t(bytes), None)
    if rc == 0:
        assert lib.fftc_set_stiffness(h, LAM.ctypes.data_as(C.c_void_p), MU.ctypes.data_as(C.c_void_p), F.FFTC_F64) == 0
    return h, rc

def solve(h, tests_to_end=5, errors_after=-1, sync_fails=0):
    rep = F.fftc_report()
    stub.stub_reset(tests_to_end, errors_after, sync_fails)
    rc = lib.fftc_solve(h, None, 1, C.byref(rep))
    stub.stub_reset(tests_to_end, -1, 0)
    return rc
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if not os.path.exists(B.OUT):
        B.build()
    out = str(tmp_path_factory.mktemp("stub") / "libhipstub.so")
    cmd = ["hipcc", "--offload-host-only", "-std=c++17", "-O1", "-shared", "-fPIC", "-nodefaultlibs", "-lstdc++", "-lc",
           "-I" + os.path.join(B.HERE, "csrc"), os.path.join(ROOT, "tests", "hip_stub.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


def _run(stub, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, stub=stub) + body], cwd=ROOT, capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]


@pytest.mark.parametrize("errors_after", [0, 1, 3, 6])
def test_failed_solve_leaves_no_queued_work(stub, errors_after):
    """A HIP error at the start, among the iterations and behind the last of them that is queued: the
    stream is waited for before the call returns."""
    _run(stub, f"""
h, rc = handle()
assert rc == 0
assert solve(h, 50, {errors_after}) == F.FFTC_E_HIP
assert stub.stub_drained()
assert solve(h) != F.FFTC_E_HIP          # the handle is usable again
""")


def test_slot_of_a_stream_that_cannot_be_waited_for_is_not_used_again(stub):
    _run(stub, """
a, _ = handle(); solve(a); wa = stub.stub_word()
F.fftc_destroy(a)
b, _ = handle(); solve(b)
assert stub.stub_word() == wa            # a returned slot is taken again
assert solve(b, 50, 3, 1) == F.FFTC_E_HIP
solve(b)
assert stub.stub_word() not in (None, wa)
F.fftc_destroy(b)
c, _ = handle(); solve(c)
assert stub.stub_word() not in (None, wa)
""")


def test_slots_of_many_handles(stub):
    """Slots over three slabs are distinct; slabs go with their last slot, except the first."""
    _run(stub, """
hs, words = [], []
for k in range(130):
    h, _ = handle((4, 4, 4)); solve(h)
    hs.append(h); words.append(stub.stub_word())
assert len(set(words)) == 130 and min(abs(x - y) for x, y in zip(sorted(words), sorted(words)[1:])) >= 128
assert stub.stub_slabs() == 3
for k in list(range(129, 127, -1)) + list(range(0, 128, 3)):
    F.fftc_destroy(hs[k])
assert stub.stub_slabs() == 2            # the third slab held the last two
again = []
for k in range(20):
    h, _ = handle((4, 4, 4)); solve(h)
    again.append(h); assert stub.stub_word() in words[0:128:3]
for h in again + [hs[k] for k in range(128) if k % 3]:
    F.fftc_destroy(h)
assert stub.stub_slabs() == 1
""")


@pytest.mark.parametrize("n", [(20, 22, 26), (16, 16, 16), (64, 50, 8)])
@pytest.mark.parametrize("prec", [0, 1])
def test_workspace_sized_before_the_boundary_table(stub, n, prec):
    """The default table has one transform type an axis, this one three: the size asked for first is
    accepted, and only a size without the fields is not."""
    _run(stub, f"""
n, prec = {n}, {prec}
bc = np.zeros((3, 3, 2), np.int8)
bc[0, :, 0] = 1; bc[1, :, :] = 1         # x, y, z axes: DCT3 or DST3, DST1 and DCT1
h = F.fftc_create(n, prec); early = F.fftc_workspace_bytes(h); F.fftc_destroy(h)
h, rc = handle(n, prec, bc, early); assert rc == 0
assert F.fftc_workspace_bytes(h) > early
assert solve(h) != F.FFTC_E_HIP
N = [v + 1 for v in n]; fields = 3 * N[0] * N[1] * N[2] * (80 if prec == 0 else 64)
assert handle(n, prec, bc, fields)[1] == F.FFTC_E_WORKSPACE
""")
