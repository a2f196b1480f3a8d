"""vr_pairs_dim2 at the limits of the links among more than 66 vertices, where
one link may pass them: 64 and 65 vertices, 64 edges outside a forest and more.
Bit-exact against the oracle; and past a limit the reduction starts without
the kernels that follow the links."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _suspension(edges, m, lone):
    """The graph `edges` on m vertices first, then each joined to a, then to
    b, and last ab, whose link is the graph; and `lone` vertices more."""
    n = m + 2 + lone
    v = np.random.default_rng(m).permutation(n)
    a, b, k = v[0], v[1], v[2:m + 2]
    e = [(k[x], k[y]) for x, y in edges] + [(a, x) for x in k] + [(b, x) for x in k] + [(a, b)]
    M = np.full((n, n), 10 ** 6, np.int32)
    for q, (x, y) in enumerate(e):
        M[x, y] = M[y, x] = q + 1
    return M, len(e) + 1


def _cycle(m):
    return [(i, (i + 1) % m) for i in range(m)]


def _bipartite(p, q):
    return [(i, p + j) for i in range(p) for j in range(q)]


CASES = [("cycle 63", _cycle(63), 63, True), ("cycle 64", _cycle(64), 64, True), ("cycle 65", _cycle(65), 65, False),
         ("cycle 129", _cycle(129), 129, False), ("bipartite 9 9", _bipartite(9, 9), 18, True),
         ("bipartite 9 10", _bipartite(9, 10), 19, False), ("bipartite 2 62", _bipartite(2, 62), 64, True),
         ("bipartite 3 40", _bipartite(3, 40), 43, False)]


@pytest.mark.parametrize("name,edges,m,fits", CASES, ids=[c[0] for c in CASES])
def test_limits(name, edges, m, fits):
    import torch
    from torch.profiler import ProfilerActivity, profile

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] links of {name}", flush=True)
    M, tau = _suspension(edges, m, 70)
    thr = ("sqdist", tau, 0)
    f = orc.build_matrix(M, thr)
    tets = orc.tetra_list(f)
    q_low = orc.reduce_dim2(f, tets, "cohomology", orc.reduce(f, "cohomology").t_low)
    want = np.full(f.T, -1, np.int64)
    want[q_low[q_low >= 0]] = np.nonzero(q_low >= 0)[0]
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), thr, maxdim=3)
    e_low, _ = vr.pairs_dim0(r)
    toe = vr.pairs_dim1(r, e_low)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        tt = vr.pairs_dim2(r, toe)
        torch.cuda.synchronize()
    r.free()
    assert np.array_equal(tt.cpu().numpy(), want)
    ran = {k.key.split("(")[0] for k in p.key_averages()}
    if not any("k_lk_pairs" in k for k in ran):
        pytest.skip("the profiler saw no kernels")
    # a long link is known before the second kernel, a link of many cycles before the reduction's last
    assert any("k_rd_round" in k for k in ran) == (not fits)
    if m > 64:
        assert not any("k_lk_reduce" in k for k in ran)
