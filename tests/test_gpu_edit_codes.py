"""The edit encoding where its kernels change path: codes longer than the
decoder's lookup table (10 bits) up to the length limit, entry counts around
the compaction's 4-entry groups and blocks, and more compaction blocks than
one piece of the prefix sum (8192); byte for byte against the reference."""
import numpy as np
import pytest

import test_gpu_edits as edits

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

msz = edits.msz


def _fibonacci(n):
    f = [1, 1]
    while len(f) < n:
        f.append(f[-1] + f[-2])
    return f


@pytest.mark.parametrize("value_syms,gap_syms", [(9, 3), (13, 5), (24, 13)])
def test_long_codes(msz, value_syms, gap_syms):
    """Fibonacci counts make the code lengths run from 1 to the number of
    symbols less one (limited to 20)."""
    rng = np.random.default_rng(101)
    exps = rng.permutation(np.repeat(np.arange(value_syms), _fibonacci(value_syms)))
    values = -np.ldexp(1.0 + rng.uniform(0.0, 0.999, exps.size), (-exps - 1).astype(np.int32)).astype(np.float32)
    counts = _fibonacci(gap_syms)[::-1]  # short gaps often, long ones rarely
    b = rng.permutation(np.repeat(np.arange(gap_syms), counts))
    gaps = (1 << np.resize(b, exps.size)) + rng.integers(0, 1 << 20, exps.size) % (1 << np.resize(b, exps.size))
    idx = np.cumsum(gaps)
    x = np.zeros(int(idx[-1]) + 5, dtype=np.float32)
    x[idx] = values
    edits._check(msz, x)


@pytest.mark.parametrize("n", [2, 3, 4, 1023, 1024, 1025, 4095, 4096, 8195, 8193 * 4096 + 6])
def test_entry_counts(msz, n):
    rng = np.random.default_rng(n % 1000)
    x = np.zeros(n, dtype=np.float32)
    at = rng.choice(n, size=min(n, 3000), replace=False)
    x[at] = -rng.exponential(1e-3, at.size).astype(np.float32)
    x[n - 1] = -1.0
    edits._check(msz, x)
