"""The network's kernels at the edges of their tiles: sides one below, at and
one above the tiles of the convolutions (16 x 8 x 8; 2D 16 x 32), of the
weight gradients (16 x 8 x 4; 2D 16 x 16) and of the features (32 x 8 columns,
16 planes), against the oracle with the bounds of test_gpu_net."""
import numpy as np
import pytest

import test_gpu_net as net

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

msz = net.msz

SHAPES = [(17, 9, 33), (16, 8, 32), (4, 7, 17), (5, 8, 15), (33, 3, 2), (1, 33, 16), (1, 16, 17), (1, 1, 31)]


@pytest.mark.parametrize("shape", SHAPES)
def test_features_at_tile_edges(msz, shape):
    net.test_features_match_oracle(msz, shape)


@pytest.mark.parametrize("shape", SHAPES)
def test_forward_at_tile_edges(msz, shape):
    net.test_forward_layers_match_oracle(msz, shape)


@pytest.mark.parametrize("shape", [(5, 9, 17), (4, 8, 16), (1, 17, 33), (9, 20, 40)])
def test_gradients_at_tile_edges(msz, shape):
    """Every gradient element within the per-element bound (the last shape
    sums the partials of many blocks)."""
    _, _, _, x = net.feature_case(shape, 14)
    params = net.random_params(15)
    rng = np.random.default_rng(16)
    t = rng.uniform(0.5, 2.0, size=shape).astype(np.float32)
    t[rng.uniform(size=shape) < 0.6] = 0.0
    flat = torch.from_numpy(net.flat_params(params)).cuda()
    feat = net.to_dev_feat(x)
    _, g = msz.net_gradients(flat, feat, torch.from_numpy(t.ravel()).cuda(), shape, edit_weight=4.0)
    got = net.unflat_grads(g.cpu().numpy())
    p, a1, a2 = msz.net_forward(flat, feat, shape, hidden=True)
    acts = [net.bits_to_float(a.cpu().numpy()).T.reshape((16,) + shape) for a in (a1, a2)]
    bounds = net._layerwise_gradient_bounds(x, params, *acts, p.cpu().numpy().reshape(shape), t, 4.0)
    for li, (dW, db, bW, bb) in enumerate(bounds):
        assert np.all(np.abs(got[li][0] - dW) <= bW), li
        assert np.all(np.abs(got[li][1] - db) <= bb), li
