"""Corrections on both sides of the rules that choose a field's grid and
direction tiles: at most 256 work items per operation (64 x 16 direction
tiles in 2D, 64 x 16 columns of 4 planes in 3D), and 512 columns of 16 planes
in 3D; one field, without allocation, and in a batch, against the oracle bit
for bit."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# 256 and 264 direction tiles; 256 and 264 columns of 4 planes; 496 and 512 columns of 16
SHAPES = [(512, 512), (513, 512), (64, 128, 128), (64, 129, 66), (256, 496, 2), (256, 512, 2)]


@pytest.fixture(scope="module")
def msz():
    import paper_2406_09423_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


@pytest.mark.parametrize("shape", SHAPES)
def test_fix_beside_the_grid_rules(msz, shape):
    rng = np.random.default_rng(31)
    f = synth.gaussian_random_field(shape, 3.0, rng).astype(np.float32)
    xi = synth.xi_for(f, 3e-3)
    fh = synth.quantize(f, xi)
    want = oracle.fix(f, fh, xi)
    df, dh = torch.from_numpy(f).cuda(), torch.from_numpy(np.ascontiguousarray(fh)).cuda()
    runs = [msz.fix(df, dh, xi, count_init=True), msz.fix_noalloc(df, dh, xi, count_init=True, g_out=torch.empty_like(df))]
    runs += msz.fix_batch([(df, dh, float(xi))] * 2, count_init=True)[1]
    for rc, d, g, st in runs:
        assert rc == want[0] and st == want[3]
        assert np.array_equal(g.cpu().numpy().view(np.uint32), want[2].view(np.uint32))
        assert np.array_equal(d.cpu().numpy().view(np.uint32), want[1].view(np.uint32))
