"""Runs of sparse C rounds (one block works through the rounds once few cases
are left): the round cap at every round, so that a run is cut anywhere;
numbers of cases around the limits at which a run starts and at which a
growing round ends it; a stall inside a run; and fields whose cases are all
sparse, alone and in a batch, against the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def msz():
    import paper_2406_09423_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _bits(a):
    return np.asarray(a.cpu() if hasattr(a, "cpu") else a, dtype=np.float32).view(np.uint32)


def _same(msz, f, fh, xi, merged, **kw):
    want = oracle.fix(f, fh, xi, merged_c=merged, **kw)
    rc, d, g, st = msz.fix(_dev(f), _dev(fh), xi, merged=merged, count_init=True, **kw)
    assert rc == want[0]
    assert np.array_equal(_bits(g), _bits(want[2])) and np.array_equal(_bits(d), _bits(want[1]))
    assert st == want[3]
    return st


@pytest.mark.parametrize("merged", [False, True])
def test_cap_at_every_round(msz, merged):
    f, fh, xi = synth.bumps128()[0]
    st = _same(msz, f, fh, xi, merged)
    rounds = sum(st["rounds"]) + st["rounds_r"]
    for cap in range(1, rounds + 2):
        _same(msz, f, fh, xi, merged, max_rounds=cap)


def _noisy(shape, share, seed, amp):
    """A ramp (no extremum inside) with lone perturbed vertices: about
    share * n false critical points of the perturbed field."""
    rng = np.random.default_rng(seed)
    f = np.add.outer(np.zeros(shape[:-1]), np.arange(shape[-1])).astype(np.float32)
    f += sum(np.arange(s, dtype=np.float32).reshape([-1 if a == k else 1 for a in range(len(shape))]) * 0.37
             for k, s in enumerate(shape[:-1]))
    fh = f + np.where(rng.uniform(size=shape) < share, amp * rng.choice([-1.0, 1.0], size=shape), 0.0)
    fh = fh.astype(np.float32)
    return f, fh, np.float32(np.abs(f.astype(np.float64) - fh).max() * 1.0001)


# about half the perturbed vertices are cases: shares on both sides of the
# limits (2D 256 and merged 151, 3D 208 and merged 72)
@pytest.mark.parametrize("shape", [(90, 110), (21, 23, 25)])
@pytest.mark.parametrize("cases", [40, 72, 150, 208, 256, 400])
@pytest.mark.parametrize("merged", [False, True])
def test_numbers_of_cases(msz, shape, cases, merged):
    n = int(np.prod(shape))
    f, fh, xi = _noisy(shape, cases / n, cases, 2.3)
    _same(msz, f, fh, xi, merged)


def _stalling():
    """Two neighbours whose float32 floors collide (f_1 < f_0, L_1 == L_0, the
    larger id above), with a longer chain of edits beside them."""
    f0, f1, xi = np.float32(0.5 + 2.0 ** -23), np.float32(0.5 + 2.0 ** -24), np.float32(4.5)
    f = np.array([[f0, f1, -3.0, -2.5, -3.5, -4.0, -4.5]], np.float32)
    L = oracle.lower_bound(f, xi)
    return f, np.array([[L[0, 0], 0.0, -3.0, -2.5, -1.0, -4.0, -4.5]], np.float32), xi


@pytest.mark.parametrize("merged", [False, True])
def test_stall(msz, merged):
    f, fh, xi = _stalling()
    assert oracle.fix(f, fh, xi, merged_c=merged)[0] == oracle.ESTALL
    _same(msz, f, fh, xi, merged)


@pytest.mark.parametrize("merged", [False, True])
def test_sparse_fields_in_a_batch(msz, merged):
    fields = [synth.bumps128(k)[0] for k in range(3)]
    fields += [_noisy((12, 14, 17), 0.02, 5, 2.3), _noisy((60, 9), 0.1, 6, 1.7), _noisy((30, 31, 32), 0.003, 8, 2.3)]
    rc, res = msz.fix_batch([(_dev(f), _dev(fh), float(xi)) for f, fh, xi in fields], merged=merged, count_init=True)
    assert rc == msz.OK
    for (f, fh, xi), (_, d, g, st) in zip(fields, res):
        want = oracle.fix(f, fh, xi, merged_c=merged)
        assert np.array_equal(_bits(g), _bits(want[2])) and st == want[3]
