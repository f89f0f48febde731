"""Labels at the edges of the label tiles (128 x 32 in 2D, 64 x 8 x 8 in 3D):
sides one below, at and one above a tile and just past two, on smooth fields
(long in-tile paths and exits through every face) and on plateaus (ties by
id), against the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(31, 127), (32, 128), (33, 129), (65, 257), (1, 300), (70, 1),
          (7, 7, 63), (8, 8, 64), (9, 9, 65), (17, 16, 130), (20, 1, 3), (1, 17, 66)]


@pytest.fixture(scope="module")
def msz():
    import paper_2406_09423_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


@pytest.mark.parametrize("shape", SHAPES)
def test_labels_at_tile_edges(msz, shape):
    rng = np.random.default_rng(91)
    smooth = synth.gaussian_random_field(shape, 4.0, rng).astype(np.float32)
    ramp = np.arange(smooth.size, dtype=np.float32).reshape(shape)  # one path through every tile
    for h in (smooth, np.round(smooth * 6).astype(np.float32), ramp, -ramp):
        M, m = msz.labels(torch.from_numpy(np.ascontiguousarray(h)).cuda())
        want_M, want_m = oracle.labels(h)
        assert np.array_equal(M.cpu().numpy().reshape(-1), np.asarray(want_M).reshape(-1))
        assert np.array_equal(m.cpu().numpy().reshape(-1), np.asarray(want_m).reshape(-1))
