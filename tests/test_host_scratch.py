"""The host side of the library on a stand-in for the HIP runtime
(fake_hip.cpp), without a GPU: where the scratch of a call comes from, what a
call does when memory is short, and the grids it launches."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PREAMBLE = """
import ctypes, sys
sys.path.insert(0, sys.argv[2])
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # ahead of the library's own runtime
fake.fake_set.argtypes = [ctypes.c_size_t, ctypes.c_int, ctypes.c_int]
fake.fake_log.restype = ctypes.c_char_p
fake.fake_live.restype = ctypes.c_size_t
import paper_2406_09423_amd as msz
L = msz.lib()
EVERY = 2 ** 63
STREAM = 4096  # the handle of a stream; never looked into
def log():
    return fake.fake_log().decode().split("\\n")[:-1]
def array(nbytes):
    a = (ctypes.c_char * (nbytes + 16))()
    keep.append(a)
    return (ctypes.addressof(a) + 15) & ~15
keep = []
n = 300 * 200
d = msz.dims_of((200, 300))
f, M, m = array(4 * n), array(4 * n), array(4 * n)
counts = msz.FalseCounts()
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-o", out, os.path.join(HERE, "fake_hip.cpp")], check=True)
    return out


def run(fake, code):
    r = subprocess.run([sys.executable, "-c", PREAMBLE + code, fake, ROOT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_labels_with_little_memory(fake):
    """Labels take one byte of scratch per vertex."""
    run(fake, """
fake.fake_set(2 * n, 0, 0)
assert L.msz_labels(f, d, M, m, None) == msz.OK
assert fake.fake_live() == 1  # the pinned counters
""")


def test_calls_after_one_without_memory(fake):
    """A call that found no memory says so, and the next one is not affected."""
    run(fake, """
opt, st = msz.Options(), msz.Stats()
opt.workspace, opt.workspace_bytes = array(L.msz_workspace_bytes(d)), L.msz_workspace_bytes(d)
fake.fake_set(100, 0, 0)  # no memory for the control block
assert L.msz_fix(f, f, d, ctypes.c_float(0.5), M, ctypes.byref(opt), ctypes.byref(st), None) == msz.ENOMEM
fake.fake_set(EVERY, 0, 0)
assert L.msz_labels(f, d, M, m, None) == msz.OK
for call in (lambda: L.msz_count_false(f, f, d, ctypes.byref(counts), None), lambda: L.msz_labels(f, d, M, m, None)):
    fake.fake_set(100, 0, 0)
    assert call() == msz.ENOMEM
    fake.fake_set(EVERY, 0, 0)
    assert call() == msz.OK
""")


def test_scratch_lies_on_the_device_of_the_stream(fake):
    """A call on a stream of another device than the current one takes its
    scratch there; on the null stream, from the current device."""
    run(fake, """
size = ctypes.c_size_t()
edits, blob = array(4 * n), array(L.msz_edits_bound(n))
feat, p = array(32 * n), array(4 * n)
params = array(4 * msz.NET_PARAMS)
for stream, device in ((STREAM, 3), (None, 1)):
    for call in (lambda: L.msz_labels(f, d, M, m, stream), lambda: L.msz_count_false(f, f, d, ctypes.byref(counts), stream),
                 lambda: L.msz_encode_edits(edits, n, blob, L.msz_edits_bound(n), ctypes.byref(size), None, stream),
                 lambda: L.msz_decode_edits(blob, size.value, edits, n, stream),
                 lambda: L.msz_net_forward(params, feat, d, p, None, None, None, 0, stream)):
        fake.fake_set(EVERY, 1, 3)
        call()
        asked = [x for x in log() if x.startswith(("pool", "default"))]
        assert asked and all(x.startswith("pool %d " % device) for x in asked), asked
""")


@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 2 ** 28), (1, 2 ** 27, 1), (2 ** 27, 1, 1), (4096, 4096, 8)])
def test_feature_grids_can_be_launched(fake, nx, ny, nz):
    """Fewer than 2^32 threads, also where a field is one vertex wide."""
    run(fake, f"""
fake.fake_pattern(1)  # a value range of 1
rc = L.msz_net_features(f, f, msz.Dims(3, {nx}, {ny}, {nz}), ctypes.c_float(0.1), array(16), None, 0, None)
assert rc == msz.OK, (rc, log())
""")


@pytest.mark.parametrize("n,some", [(3600 * 2400, (600000, 700000, 840001, 8000000)), (2 ** 27 + 5, (9000000, 11000001, 16000000)),
                                    (300 * 200, (4100, 5400, 6100, 8000))])
def test_new_edits_need_no_new_memory(fake, n, some):
    """The scratch of an encoding is of the same size for any edits of a field
    (of a large field, or of few edits, for edits of about the same number), so
    that the pool has it at hand."""
    run(fake, f"""
size = ctypes.c_size_t()
asked = []
for m in {some}:
    fake.fake_set(EVERY, 0, 0)
    fake.fake_word(m)  # the number of edits, and the words of the stream
    rc = L.msz_encode_edits(f, {n}, M, ctypes.c_size_t(2 ** 40), ctypes.byref(size), None, None)
    assert rc == msz.OK, rc
    asked.append([x for x in log() if x.startswith(("pool", "default"))])
assert all(a == asked[0] for a in asked), asked
""")


@pytest.mark.parametrize("nx,ny,blocks", [(120, 130, 256), (3600, 2400, 1024)])
def test_timed_corrections_launch_the_same_grids(fake, nx, ny, blocks):
    """What a timed run of a field measures is what an untimed one runs: the
    blocks of its steps do not depend on the timing."""
    run(fake, f"""
st = msz.Stats()
for flags in (0, msz.FLAG_TIMING, 0):
    fake.fake_set(EVERY, 0, 0)
    opt = msz.Options()
    opt.flags = flags
    rc = L.msz_fix(f, f, msz.Dims(2, {nx}, {ny}, 1), ctypes.c_float(0.5), M, ctypes.byref(opt), ctypes.byref(st), None)
    assert rc == msz.OK, rc
    steps = [x for x in log() if x.startswith("step")]
    assert steps and all(x == "step {blocks}" for x in steps), steps
""")
