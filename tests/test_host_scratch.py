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
fake.fake_live_bytes.restype = ctypes.c_size_t
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
assert fake.fake_live_bytes() < 2 << 20
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
fake.fake_set(100, 0, 0)  # nor for scratch
assert L.msz_count_false(f, f, d, ctypes.byref(counts), None) == msz.ENOMEM
fake.fake_set(EVERY, 0, 0)
assert L.msz_labels(f, d, M, m, None) == msz.OK
assert L.msz_count_false(f, f, d, ctypes.byref(counts), None) == msz.OK
""")


def test_scratch_lies_on_the_device_of_the_stream(fake):
    """A call takes kept scratch of its stream's device only; on the null
    stream, of the current device."""
    run(fake, """
size = ctypes.c_size_t()
edits, blob = array(4 * n), array(L.msz_edits_bound(n))
feat, p = array(32 * n), array(4 * n)
params = array(4 * msz.NET_PARAMS)
for k, call in enumerate([
        lambda s: L.msz_labels(f, d, M, m, s), lambda s: L.msz_count_false(f, f, d, ctypes.byref(counts), s),
        lambda s: L.msz_encode_edits(edits, n, blob, L.msz_edits_bound(n), ctypes.byref(size), None, s),
        lambda s: L.msz_decode_edits(blob, size.value, edits, n, s),
        lambda s: L.msz_net_forward(params, feat, d, p, None, None, None, 0, s)]):
    a, b = 2 * k, 2 * k + 1  # devices not used yet
    asked = []
    for stream, current, of_stream in ((STREAM, a, b), (STREAM, a, b), (None, a, b), (None, b, a), (STREAM, b, a)):
        fake.fake_set(EVERY, current, of_stream)
        call(stream)
        asked.append(any(x.startswith("device") for x in log()))
    assert asked == [True, False, True, False, False], asked
""")


def test_scratch_is_kept_and_bounded(fake):
    """Calls of different sizes in turn take what earlier ones left; what is
    kept stays below 512 MB, and is given back when memory is short."""
    run(fake, """
def call(nx, ny):
    fake.fake_set(EVERY, 0, 0)
    assert L.msz_count_false(f, f, msz.Dims(2, nx, ny, 1), ctypes.byref(counts), STREAM) == msz.OK
    return [x for x in log() if x.startswith("device")]
sizes = [(3600, 2400), (300, 200), (1800, 1200), (3600, 2390), (320, 190)]
for nx, ny in sizes:
    call(nx, ny)
assert not any(call(nx, ny) for nx, ny in sizes)
assert fake.fake_live_bytes() < 512 << 20
for k in range(12):
    call(5000 + 700 * k, 1000)
    assert fake.fake_live_bytes() <= (512 << 20) + (1 << 20)
    call(500, 1000 + 500 * k)
big = 30000 * 3000  # 900 MB of scratch: not kept
assert call(30000, 3000) and call(30000, 3000)
assert fake.fake_live_bytes() <= (512 << 20) + (1 << 20)
fake.fake_set(30 << 20, 0, 0)  # a request above 30 MB fails: everything kept is given back
assert L.msz_count_false(f, f, msz.Dims(2, 30000, 3000, 1), ctypes.byref(counts), STREAM) == msz.ENOMEM
assert fake.fake_live_bytes() <= 1 << 20
""")


@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 2 ** 28), (1, 2 ** 27, 1), (2 ** 27, 1, 1), (4096, 4096, 8)])
def test_feature_grids_can_be_launched(fake, nx, ny, nz):
    """Fewer than 2^32 threads, also where a field is one vertex wide."""
    run(fake, f"""
fake.fake_pattern(1)  # a value range of 1
rc = L.msz_net_features(f, f, msz.Dims(3, {nx}, {ny}, {nz}), ctypes.c_float(0.1), array(16), None, 0, None)
assert rc == msz.OK, (rc, log())
""")


@pytest.mark.parametrize("n,some", [(3600 * 2400, (600000, 700000, 640001, 1, 690000)),
                                    (2 ** 27 + 5, (9000000, 11000001, 10500000)), (300 * 200, (4100, 8000, 60000))])
def test_new_edits_need_no_new_memory(fake, n, some):
    """Encoding edits of about as many as before takes no new memory."""
    run(fake, f"""
size = ctypes.c_size_t()
asked = []
for k, m in enumerate((max({some}),) + {some}):
    fake.fake_set(EVERY, 0, 0)
    fake.fake_word(m)  # the number of edits, and the words of the stream
    rc = L.msz_encode_edits(f, {n}, M, ctypes.c_size_t(2 ** 40), ctypes.byref(size), None, None)
    assert rc == msz.OK, rc
    assert k == 0 or not [x for x in log() if x.startswith("device")], (m, log())
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
