"""Network features of flat and tall grids, whose columns are dealt to blocks in
tiles of 128 x 2, 4 x 64, 256 x 1 and 1 x 256 instead of 32 x 8, against the oracle."""
import numpy as np
import pytest

import oracle
import oracle.net_ref as nr

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# (nz, ny, nx): on both sides of the rule, and at the edges of the tiles
@pytest.mark.parametrize("shape", [(1, 1, 300), (1, 2, 128), (1, 3, 129), (20, 2, 257), (1, 256, 1), (2, 515, 1), (18, 1, 256), (1, 3, 2), (1, 64, 4), (17, 65, 5),
                                   (1, 129, 16), (3, 130, 24), (33, 1, 1), (2, 9, 33)])
def test_features_of_flat_and_tall_grids(shape):
    import paper_2406_09423_amd as msz
    xi = 0.01
    rng = np.random.default_rng(5)
    f = rng.uniform(0, 1, size=shape).astype(np.float32)
    fh = (f + rng.uniform(-xi, xi, size=shape)).astype(np.float32)
    bits = oracle.case_flags(f, fh) if shape[0] > 1 else oracle.case_flags(f[0], fh[0])[None]
    x = nr.features(f, fh, xi, bits & 15, float(f.max()) - float(f.min()), oracle.dirs(f), oracle.dirs(fh))
    ref = nr.bf16(x).reshape(12, -1).T
    got = msz.net_features(torch.from_numpy(f).cuda(), torch.from_numpy(fh).cuda(), xi).cpu().numpy()
    g = (got.view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    for c in range(12):
        # the box-mean channels: one BF16 ulp, as sums in another order may round differently
        tol = 2.0 ** -7 * np.abs(ref[:, c]) + 1e-30 if c in (0, 7) else 0.0
        assert np.all(np.abs(g[:, c] - ref[:, c]) <= tol), c
    assert np.all(g[:, 12:] == 0)
