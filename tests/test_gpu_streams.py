"""Builds on several streams at once, from a thread each: sorts and scans whose
work-groups wait for one another, more of them together than the device holds.
Each equals the build alone, and every one ends."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _cloud(n, q, seed):
    """n points, and a squared distance that about q of their pairs stay below."""
    p = np.random.default_rng(seed).integers(-15000, 15001, (n, 3)).astype(np.int16)
    s = p[np.random.default_rng(1).integers(0, n, (2, 20000))].astype(np.int64)
    d = np.sort(((s[0] - s[1]) ** 2).sum(1))
    return p, ("sqdist", int(d[int(len(d) * q / (n * (n - 1) / 2))]), 0)


@pytest.mark.parametrize("shapes", [
    [(8192, 1400000)] * 6,                                       # 16384 tiles of pairs, under 768 kept
    [(8192, 1400000), (2000, 300000), (1400, 400000)] * 2,      # with sorts of few tiles
])
def test_streams(shapes):
    import torch

    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    jobs = []
    for i, (n, q) in enumerate(shapes):
        p, thr = _cloud(n, q, i)
        x = torch.from_numpy(p).to("cuda:0")
        r = vr.build(x, thr)
        assert r.K > q // 2 and r.K <= 768 * 2048
        jobs.append((x, thr, (r.edge_ij().clone(), r.edge_q().clone(), r.tri_key().clone())))
        r.free()
    torch.cuda.synchronize()
    bad = []

    def work(i):
        x, thr, want = jobs[i]
        with torch.cuda.stream(torch.cuda.Stream()):
            for k in range(6):
                r = vr.build(x, thr)
                got = (r.edge_ij(), r.edge_q(), r.tri_key())
                if not all(torch.equal(a, b) for a, b in zip(got, want)):
                    bad.append((i, k))
                del got
                r.free()
                print(f"[gpu] stream {i} build {k}", flush=True)

    t = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for x in t:
        x.start()
    for x in t:
        x.join()
    assert not bad
