"""Calls on a workspace of exactly the size that is asked for write nothing
past its end, and give the results of calls without a workspace."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _guarded(nbytes):
    buf = torch.full((nbytes + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    return buf[:nbytes], buf[nbytes:]


# a few vertices (all small arrays packed), and grids with more tiles of the
# weight gradient than partial sums
@pytest.mark.parametrize("shape", [(1, 1), (3, 5), (8, 8), (1, 300), (128, 128), (4, 6, 5), (31, 33, 35)])
def test_workspace_of_the_asked_size(shape):
    import paper_2406_09423_amd as msz
    rng = np.random.default_rng(3)
    f = rng.uniform(0, 1, size=shape).astype(np.float32)
    xi = np.float32(0.05)
    fd, fhd = torch.from_numpy(f).cuda(), torch.from_numpy(synth.quantize(f, xi)).cuda()
    ws, guard = _guarded(msz.workspace_bytes(shape))
    got, want = msz.fix(fd, fhd, xi, workspace=ws, count_init=True), msz.fix(fd, fhd, xi, count_init=True)
    assert got[0] == want[0] and got[3] == want[3] and torch.equal(got[2], want[2])
    assert bool((guard == 0xA5).all())
    ws, guard = _guarded(msz.net_workspace_bytes(shape))
    feat = torch.from_numpy(rng.uniform(-1, 1, (f.size, 16)).astype(np.float32)).cuda().bfloat16().view(torch.int16)
    params = torch.from_numpy(rng.uniform(-0.2, 0.2, msz.NET_PARAMS).astype(np.float32)).cuda()
    t = torch.from_numpy((rng.uniform(size=f.size) < 0.3).astype(np.float32)).cuda()
    (l0, g0), (l1, g1) = (msz.net_gradients(params, feat, t, shape, edit_weight=2.0, workspace=w) for w in (ws, None))
    assert l0 == l1 and torch.equal(g0, g1)
    assert bool((guard == 0xA5).all())
