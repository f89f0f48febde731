"""Corrections of fields whose sides lie one below, at and one above the tiles
(label tiles 128 x 32 and 64 x 8 x 8, direction tiles 64 x 16 and 64 x 16
columns) and whose rows start at every alignment, alone and in a batch, both
C schedules, against the oracle bit for bit (the start field's mislabelled
vertices included, which resolves every vertex's labels)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(31, 127), (33, 129), (64, 128), (65, 258), (16, 64), (17, 65), (15, 63), (40, 1), (1, 130),
          (7, 7, 63), (9, 9, 65), (8, 8, 64), (17, 16, 130), (16, 17, 66), (33, 18, 67), (5, 40, 3), (2, 1, 70)]


@pytest.fixture(scope="module")
def msz():
    import paper_2406_09423_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def _field(shape, seed, rel):
    rng = np.random.default_rng(seed)
    f = synth.gaussian_random_field(shape, 3.0, rng).astype(np.float32)
    f = (f + np.float32(2e-3) * rng.standard_normal(shape)).astype(np.float32)
    xi = synth.xi_for(f, rel)
    return f, synth.quantize(f, xi), xi


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _bits(a):
    return np.asarray(a.cpu() if hasattr(a, "cpu") else a, dtype=np.float32).view(np.uint32)


def _check(res, want):
    rc, d, g, st = res
    assert rc == want[0] and st == want[3]
    assert np.array_equal(_bits(g), _bits(want[2])) and np.array_equal(_bits(d), _bits(want[1]))


@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_fix_at_tile_edges(msz, shape, merged):
    f, fh, xi = _field(shape, 7, 1e-2)
    _check(msz.fix(_dev(f), _dev(fh), xi, merged=merged, count_init=True), oracle.fix(f, fh, xi, merged_c=merged))


@pytest.mark.parametrize("merged", [False, True])
def test_batch_at_tile_edges(msz, merged):
    fields = [_field(shape, 20 + k, (1e-2, 3e-2)[k % 2]) for k, shape in enumerate(SHAPES)]
    _, res = msz.fix_batch([(_dev(f), _dev(fh), float(xi)) for f, fh, xi in fields], merged=merged, count_init=True)
    for (f, fh, xi), r in zip(fields, res):
        _check(r, oracle.fix(f, fh, xi, merged_c=merged))
