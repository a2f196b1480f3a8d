"""vr_pairs_dim1 where no edge is critical (ultrametrics, paths along a tree)
and where one cycle among such points makes one.  Bit-exact against the
oracle; and where none is, the links of the edges are not gone through."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _ultrametric(n):
    x = np.arange(n)[:, None] ^ np.arange(n)[None]
    return np.where(x > 0, np.floor(np.log2(np.maximum(x, 1))).astype(np.int64) + 1, 0).astype(np.int32)


def _tree(n, seed):
    g = np.random.default_rng(seed)
    M = np.zeros((n, n), np.int32)
    for v in range(1, n):
        u = g.integers(0, v)
        M[v, :v] = M[:v, v] = M[u, :v] + g.integers(1, 50)
    return M


def _with_cycle(M, k):
    """k more points, a cycle of edges of length 1, far from the others."""
    n = len(M)
    C = np.abs(np.arange(k)[:, None] - np.arange(k)[None])
    W = np.full((n + k, n + k), int(M.max()) + k, np.int32)
    W[:n, :n] = M
    W[n:, n:] = np.minimum(C, k - C)
    return W


CASES = {"ultrametric 64": _ultrametric(64), "ultrametric 150": _ultrametric(150), "tree 100": _tree(100, 5),
         "tree 3": _tree(3, 1), "ultrametric and cycle": _with_cycle(_ultrametric(100), 12),
         "tree and cycle": _with_cycle(_tree(90, 7), 5)}


@pytest.mark.parametrize("name", list(CASES))
def test_pairs(name):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] {name}", flush=True)
    M, thr = CASES[name], ("sqdist", int(CASES[name].max()) + 1, 0)
    f = orc.build_matrix(M, thr)
    p = orc.reduce(f, "cohomology")
    want = np.full(f.K, -1, np.int64)
    want[p.t_low[p.t_low >= 0]] = np.nonzero(p.t_low >= 0)[0]
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), thr)
    e_low, _ = vr.pairs_dim0(r)
    for _ in range(2):
        assert np.array_equal(vr.pairs_dim1(r, e_low).cpu().numpy().astype(np.int64), want)
    r.free()


def test_share_of_the_time():
    import torch
    from torch.profiler import ProfilerActivity, profile

    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[gpu] ultrametric 512", flush=True)
    r = vr.build_matrix(torch.from_numpy(_ultrametric(512)).to("cuda:0"), ("sqdist", 100, 0))
    e_low, _ = vr.pairs_dim0(r)
    vr.pairs_dim1(r, e_low)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        for _ in range(5):
            vr.pairs_dim1(r, e_low)
        torch.cuda.synchronize()
    r.free()
    took = {k.key: k.device_time_total for k in p.key_averages()}
    keys, links = (sum(v for k, v in took.items() if name in k) for name in ("k_mo_range", "k_mo_link"))
    if keys == 0:
        pytest.skip("the profiler saw no kernels")
    print(f"[gpu] the keys {keys / 5:.0f} us, the links {links / 5:.0f}", flush=True)
    assert links < keys
