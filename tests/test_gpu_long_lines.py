"""Labels and false counts where an integral line winds through hundreds of
label tiles (a corridor that turns back and forth through the grid, its values
rising along it, between low walls), against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(64, 1024), (63, 1001), (9, 24, 512), (10, 23, 515)]


@pytest.fixture(scope="module")
def msz():
    import paper_2406_09423_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def corridor(shape):
    """Every second row (of every second plane), joined at alternating ends."""
    h = -np.ones((1,) * (3 - len(shape)) + tuple(shape), np.float32)
    nz, ny, nx = h.shape
    rows, ys = [], list(range(0, ny, 2))
    for z in range(0, nz, 2):
        rows += [(z, y) for y in (ys if z % 4 == 0 else ys[::-1])]
    t = 0
    for k, (z, y) in enumerate(rows):
        xs = range(nx) if k % 2 == 0 else range(nx - 1, -1, -1)
        for x in xs:
            t += 1
            h[z, y, x] = t
        if k + 1 < len(rows):
            t += 1
            z1, y1 = rows[k + 1]
            h[(z + z1) // 2, (y + y1) // 2, xs[-1]] = t
    return h.reshape(shape)


@pytest.mark.parametrize("shape", SHAPES)
def test_lines_through_hundreds_of_tiles(msz, shape):
    h = corridor(shape)
    g = h.copy()
    g.reshape(-1)[np.argmax(h)] = -2.0  # the line ends one vertex earlier
    for a, b in ((h, g), (-h, -g)):
        M, m = msz.labels(torch.from_numpy(a).cuda())
        want_M, want_m = oracle.labels(a)
        assert np.array_equal(M.cpu().numpy().reshape(-1), np.asarray(want_M).reshape(-1))
        assert np.array_equal(m.cpu().numpy().reshape(-1), np.asarray(want_m).reshape(-1))
        got = msz.count_false(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda())
        want = oracle.count_false(a, b)
        for key in want:
            assert int(got[key]) == int(want[key]), key


@pytest.mark.parametrize("shape", [(65472, 128), (65504, 128), (65505, 129), (7, 9, 64 * 682), (8, 16, 64 * 1024)])
def test_counts_beside_the_tile_rule(msz, shape):
    """2046, 2047 and 4096 label tiles in 2D, 1364 and 2048 in 3D: items of a
    quarter tile below 2048 tiles, of a tile from there on."""
    rng = np.random.default_rng(17)
    f = np.round(rng.standard_normal(shape) * 8).astype(np.float32)
    g = (f + rng.integers(-1, 2, shape)).astype(np.float32)
    got = msz.count_false(torch.from_numpy(f).cuda(), torch.from_numpy(g).cuda())
    want = oracle.count_false(f, g)
    for key in want:
        assert int(got[key]) == int(want[key]), key
