"""A batch of one field runs the one-field step kernel: its results equal the
oracle's, bit for bit, on fields of several label tiles whose lines cross
them and whose correction needs troublemaker rounds."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(150, 420), (30, 31, 200)]  # 5 x 4 label tiles of 128 x 32; 4 x 4 x 4 of 64 x 8 x 8


@pytest.fixture(scope="module")
def msz():
    import paper_2406_09423_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def _field(shape):
    rng = np.random.default_rng(71)
    f = synth.gaussian_random_field(shape, 3.0 if len(shape) == 2 else 11.0 / 3.0, rng).astype(np.float32)
    xi = synth.xi_for(f, 1e-3)
    return f, synth.quantize(f, xi), xi


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _bits(a):
    return np.asarray(a.cpu() if hasattr(a, "cpu") else a, dtype=np.float32).view(np.uint32)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("count_init", [False, True])
@pytest.mark.parametrize("timing", [False, True])
def test_batch_of_one(msz, shape, merged, count_init, timing):
    f, fh, xi = _field(shape)
    want = oracle.fix(f, fh, xi, merged_c=merged)
    assert want[3]["rounds_r"] > 0
    rc, res = msz.fix_batch([(_dev(f), _dev(fh), float(xi))], merged=merged, count_init=count_init, timing=timing)
    (rc1, d, g, st), = res
    assert rc == rc1 == want[0]
    assert st == dict(want[3], mislabel_init=want[3]["mislabel_init"] if count_init else -1)
    assert np.array_equal(_bits(g), _bits(want[2])) and np.array_equal(_bits(d), _bits(want[1]))


@pytest.mark.parametrize("shape", SHAPES)
def test_batch_of_one_preemptive(msz, shape):
    f, fh, xi = _field(shape)
    rc, ((_, d, g, st),) = msz.fix_batch([(_dev(f), _dev(fh), float(xi))], preemptive=True)
    assert rc == msz.OK
    g = g.cpu().numpy()
    assert all(v == 0 for v in oracle.count_false(f, g).values())
    assert (np.abs(f.astype(np.float64) - g.astype(np.float64)) <= float(xi)).all() and (g <= fh).all()
    assert st["n_edited"] == int((g != fh).sum())
