"""Labels and false counts of smooth fields, whose integral lines run through
many label tiles: results against the oracle on both sides of the rules by which
the comparison leaves its direct walks (1024 tiles, the share of lines that
leave their tile, the length of a chain), and times beside those of a rough
field."""
import time

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def msz():
    import paper_2406_09423_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def _bumps(shape, smooth, seed):
    """A sum of wide bumps; the planes (rows) past the share `smooth` are noise."""
    rng = np.random.default_rng(seed)
    axes = np.meshgrid(*[np.linspace(0, 1, s, dtype=np.float32) for s in shape], indexing="ij", sparse=True)
    f = np.zeros(shape, np.float32)
    for _ in range(5):
        c = rng.uniform(0.1, 0.9, len(shape))
        f += np.exp(-sum((x - np.float32(a)) ** 2 for x, a in zip(axes, c)) / np.float32(0.05))
    k = int(shape[0] * smooth)
    f[k:] = rng.standard_normal((shape[0] - k,) + shape[1:])
    return f


def _seconds(call):
    call()
    times = []
    for _ in range(9):
        torch.cuda.synchronize()
        t = time.perf_counter()
        call()
        times.append(time.perf_counter() - t)
    return sorted(times)[4]


# 1088, 1280 and 1008 label tiles, and 99 and 60
@pytest.mark.parametrize("shape", [(2048, 2176), (64, 128, 640), (2000, 2048), (350, 1100), (40, 31, 150)])
@pytest.mark.parametrize("smooth", [1.0, 0.6, 0.15])
def test_smooth_and_half_smooth_fields(msz, shape, smooth):
    f = _bumps(shape, smooth, 7)
    g = f + (np.random.default_rng(8).uniform(-1, 1, shape) * 1e-3 * (np.arange(shape[-1]) % 97 == 0)).astype(np.float32)
    fd, gd = torch.from_numpy(f).cuda(), torch.from_numpy(g).cuda()
    M, m = msz.labels(fd)
    want_M, want_m = oracle.labels(f)
    assert np.array_equal(M.cpu().numpy(), want_M) and np.array_equal(m.cpu().numpy(), want_m)
    got, want = msz.count_false(fd, gd), oracle.count_false(f, g)
    assert {k: int(v) for k, v in got.items()} == {k: int(v) for k, v in want.items()}


@pytest.mark.parametrize("shape", [(2400, 3600), (256, 256, 256)])
def test_count_of_smooth_start_fields(msz, shape):
    """Counting the mislabelled vertices of the start field adds less to the
    correction of a ramp than one and a half times what it takes without
    (following every vertex's chain added two to three and a half times)."""
    f = sum(torch.linspace(0, k + 1.0, s, device="cuda").reshape([-1 if a == k else 1 for a in range(len(shape))])
            for k, s in enumerate(shape)).contiguous()
    ws = torch.empty(msz.workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    plain, counted = (_seconds(lambda: msz.fix(f, f, 0.1, workspace=ws, count_init=c)) for c in (False, True))
    assert counted < 2.5 * plain


@pytest.mark.parametrize("shape", [(350, 1100), (40, 31, 150)])
@pytest.mark.parametrize("smooth", [1.0, 0.5])
def test_mislabelled_vertices_of_smooth_start_fields(msz, shape, smooth):
    f = _bumps(shape, smooth, 9)
    fh = (f - np.random.default_rng(10).uniform(0, 1e-3, shape)).astype(np.float32)
    want = oracle.fix(f, fh, 2e-3, max_rounds=1)
    fd, fhd = torch.from_numpy(f).cuda(), torch.from_numpy(fh).cuda()
    runs = [msz.fix(fd, fhd, 2e-3, max_rounds=1, count_init=True)]
    runs += msz.fix_batch([(fd, fhd, 2e-3)] * 2, max_rounds=1, count_init=True)[1]
    for rc, d, g, st in runs:
        assert rc == want[0] and st == want[3]
        assert np.array_equal(g.cpu().numpy(), want[2])


@pytest.mark.parametrize("shape", [(2400, 3600), (256, 256, 256)])
def test_smooth_fields_take_little_longer(msz, shape):
    """A ramp's lines run through the whole grid; its labels and counts take
    less than three times those of a rough field (walking every line took seven
    to twelve times as long)."""
    gen = torch.Generator(device="cuda").manual_seed(1)
    rough = torch.randn(shape, generator=gen, device="cuda")
    ramp = sum(torch.linspace(0, k + 1.0, s, device="cuda").reshape([-1 if a == k else 1 for a in range(len(shape))])
               for k, s in enumerate(shape)).contiguous()

    for call in (lambda h: msz.labels(h), lambda h: msz.count_false(h, 2 * h)):
        assert _seconds(lambda: call(ramp)) < 3 * _seconds(lambda: call(rough))
