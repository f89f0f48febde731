"""Calls without a workspace take their scratch from the library's pool: from
several threads, each with its own stream, results equal those of one thread."""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_threads_and_streams_share_the_pool():
    import paper_2406_09423_amd as msz
    rng = np.random.default_rng(111)
    fields = []
    for k in range(4):
        f = synth.gaussian_random_field((150 + 37 * k, 211), 3.0, rng).astype(np.float32)
        xi = synth.xi_for(f, 1e-3)
        fields.append((torch.from_numpy(f).cuda(), torch.from_numpy(synth.quantize(f, xi)).cuda(), float(xi)))

    def work(k):
        f, fh, xi = fields[k]
        rc, d, g, st = msz.fix(f, fh, xi)
        assert rc == msz.OK
        M, m = msz.labels(g)
        counts = msz.count_false(f, g)
        rc, blob, _ = msz.encode_edits(d)
        assert rc == msz.OK
        rc, back = msz.decode_edits(blob, d.shape)
        assert rc == msz.OK
        return [t.cpu() for t in (d, g, M, m, blob, back)], st, counts

    want = [work(k) for k in range(4)]
    got = [None] * 4

    def run(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(5):
                got[k] = work(k)
        s.synchronize()

    threads = [threading.Thread(target=run, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(4):
        assert got[k][1:] == want[k][1:]
        for a, b in zip(got[k][0], want[k][0]):
            assert torch.equal(a, b)
