"""The workspaces a caller is asked for do not grow: a buffer of the sizes
that the library has asked for before is still accepted."""
import itertools

import pytest

import paper_2406_09423_amd as msz


def up(x, to=256):
    return (x + to - 1) // to * to


def tiles(dims, tile):
    p = 1
    for d, t in zip(dims, tile):
        p *= (d + t - 1) // t
    return p


def fix_bytes(nx, ny, nz, ndim):
    n = nx * ny * nz
    chunks = (n + 4095) // 4096
    label_tiles = tiles((nx, ny, nz), (128, 32, 1) if ndim == 2 else (64, 8, 8))
    return (6 * up(4 * n) + 2 * up(n) + 3 * up(up(n, 16)) + 2 * up(4 * chunks) + up(8 * chunks) + up(label_tiles))


def net_bytes(nx, ny, nz):
    n = nx * ny * nz
    conv_tiles = tiles((nx, ny, nz), (16, 32, 1) if nz == 1 else (16, 8, 8))
    return (2 * up(n + 16) + 5 * up(32 * n) + 3 * up(4 * n) + up(conv_tiles * 27 * 256 * 4) + up(conv_tiles * 16 * 4)
            + up(2048 * 2 * 4))


SHAPES_2D = [(1, k) for k in range(1, 1500)] + list(itertools.product((2, 7, 31, 64, 129, 500), (1, 5, 33, 128, 1025)))
SHAPES_3D = list(itertools.product((1, 2, 5, 9, 33, 64), (1, 3, 8, 21, 65), (1, 2, 17, 64, 300)))


@pytest.mark.parametrize("shapes", [SHAPES_2D, SHAPES_3D])
def test_workspaces_do_not_grow(shapes):
    for shape in shapes:
        dims = tuple(reversed(shape)) + (1,) * (3 - len(shape))
        a, b = fix_bytes(*dims, len(shape)), net_bytes(*dims)
        assert msz.workspace_bytes(shape) == a, shape
        assert msz.net_workspace_bytes(shape) <= b, shape
        assert msz.learned_workspace_bytes(shape) <= a + b, shape
