"""vr_pairs_dim0 where long runs of edges join the same two components: levels
of an ultrametric, blocks of several sizes, in the vertices' order and in a
random one, below and above the edges that are looked up again at a time.
Bit-exact against Kruskal's order; and an ultrametric takes a few times a
random order and not many."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _levels(n, base):
    a, b = np.arange(n)[:, None], np.arange(n)[None]
    M = np.zeros((n, n), np.int32)
    level = 1
    while True:
        apart = a != b
        if not apart.any():
            return M
        M[apart] = level
        a, b, level = a // base, b // base, level + 1


def _kruskal(ij, n):
    par = np.arange(n)

    def find(v):
        while par[v] != v:
            par[v] = par[par[v]]
            v = par[v]
        return v

    low = np.full(len(ij), -1, np.int64)
    for f, (a, b) in enumerate(ij):
        a, b = find(a), find(b)
        if a != b:
            low[f] = max(a, b)
            par[max(a, b)] = min(a, b)
    return low


@pytest.mark.parametrize("n,base,shuffled", [(150, 2, False), (512, 2, False), (512, 2, True), (600, 24, False), (730, 3, True),
                                             (1000, 500, False), (1000, 10, False)])
def test_levels(n, base, shuffled):
    import torch

    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] {n} points, {base} to a block, shuffled={shuffled}", flush=True)
    M = _levels(n, base)
    if shuffled:
        v = np.random.default_rng(n).permutation(n)
        M = M[v][:, v]
    r = vr.build_matrix(torch.from_numpy(np.ascontiguousarray(M)).to("cuda:0"), ("full", 0, 1))
    e_low, death = vr.pairs_dim0(r)
    low = e_low.cpu().numpy().astype(np.int64)
    want = _kruskal(r.edge_ij().cpu().numpy().reshape(-1, 2), n)
    r.free()
    assert np.array_equal(low, want)
    at = np.full(n, -1, np.int64)
    at[want[want >= 0]] = np.nonzero(want >= 0)[0]
    assert np.array_equal(death.cpu().numpy().astype(np.int64), at)


def test_time():
    import torch

    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 512
    iu = np.triu_indices(n, 1)
    W = np.zeros((n, n), np.int32)
    W[iu] = 1 + np.random.default_rng(1).permutation(len(iu[0]))
    took = []
    for name, M in (("random", W + W.T), ("ultrametric", _levels(n, 2))):
        print(f"[gpu] time of {name}", flush=True)
        r = vr.build_matrix(torch.from_numpy(np.ascontiguousarray(M)).to("cuda:0"), ("full", 0, 1))
        best = 1e9
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(10):
                vr.pairs_dim0(r)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t0) / 10)
        r.free()
        took.append(best)
    print(f"[gpu] {took[0] * 1e6:.0f} us, then {took[1] * 1e6:.0f}", flush=True)
    assert took[1] < 4 * took[0]  # 3 with the runs cut short, 5 edge by edge
