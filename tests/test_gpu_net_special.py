"""Network features of values whose quotients are not ordinary numbers: zeros
of either sign (also where the box mean is zero) and infinities in the
decompressed field, against the oracle; a difference that is not a number
clamps to -8, as the maximum of it and -8 does."""
import numpy as np
import pytest

import oracle
import oracle.net_ref as nr

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [(1, 19, 40), (9, 11, 35)])
@pytest.mark.parametrize("special", [-0.0, np.inf, -np.inf])
def test_features_of_special_values(shape, special):
    import paper_2406_09423_amd as msz
    xi = 0.01
    rng = np.random.default_rng(5)
    f = rng.uniform(0, 1, size=shape).astype(np.float32)
    fh = (f + rng.uniform(-xi, xi, size=shape)).astype(np.float32)
    if special == 0.0:  # a slab of zeros of f, of negative zeros of fhat: box means of +0 inside it
        f[:, 3:12] = 0.0
        fh[:, 3:12] = special
    else:
        fh.reshape(-1)[rng.choice(fh.size, 20, replace=False)] = special
    bits = oracle.case_flags(f, fh) if shape[0] > 1 else oracle.case_flags(f[0], fh[0])[None]
    with np.errstate(invalid="ignore"):
        x = nr.features(f, fh, xi, bits & 15, float(f.max()) - float(f.min()), oracle.dirs(f), oracle.dirs(fh))
    x[np.isnan(x)] = -8.0
    ref = nr.bf16(x).reshape(12, -1).T
    got = msz.net_features(torch.from_numpy(f).cuda(), torch.from_numpy(fh).cuda(), xi).cpu().numpy()
    g = (got.view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    for c in range(12):
        # the box-mean channels: one BF16 ulp, as sums in another order may round differently
        tol = 2.0 ** -7 * np.abs(ref[:, c]) + 1e-30 if c in (0, 7) else 0.0
        assert np.all(np.abs(g[:, c] - ref[:, c]) <= tol), c
        zero = ref[:, c] == 0
        assert np.array_equal(np.signbit(g[zero, c]), np.signbit(ref[zero, c])), c
