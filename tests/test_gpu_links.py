"""vr_pairs_dim2 from the links of the edges: random ranks (links with cycles),
cycles of up to 64 edges, many independent cycles in one link, and the
limits past which the coboundaries are reduced instead (65 vertices in a
link, more than 64 edges outside a forest).  Bit-exact against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(M, tau, label):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    thr = ("sqdist", tau, 0)
    f = orc.build_matrix(M, thr)
    tets = orc.tetra_list(f)
    p1 = orc.reduce(f, "cohomology")
    q_low = orc.reduce_dim2(f, tets, "cohomology", p1.t_low)
    want = np.full(f.T, -1, np.int64)
    want[q_low[q_low >= 0]] = np.nonzero(q_low >= 0)[0]
    print(f"[gpu] links {label} K={f.K} T={f.T} T3={len(tets)}", flush=True)
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), thr, maxdim=3)
    e_low, _ = vr.pairs_dim0(r)
    tt = vr.pairs_dim2(r, vr.pairs_dim1(r, e_low)).cpu().numpy()
    r.free()
    assert np.array_equal(tt, want)


@pytest.mark.parametrize("n,share", [(5, 1.0), (14, 1.0), (20, 0.6), (26, 0.5), (30, 0.45), (40, 0.4), (60, 0.25)])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_random_ranks(n, share, seed):
    rng = np.random.default_rng(1000 * seed + n)
    iu = np.triu_indices(n, 1)
    M = np.zeros((n, n), np.int64)
    M[iu] = 1 + rng.permutation(len(iu[0]))
    _check((M + M.T).astype(np.int32), int(len(iu[0]) * share) + 1, f"random n={n}")


def _suspension(edges, m, seed):
    """The graph `edges` on m vertices first, in random order, then each joined
    to a, then to b, and last ab, whose link is the graph."""
    rng = np.random.default_rng(seed)
    v = rng.permutation(m + 2)
    a, b, k = v[0], v[1], v[2:]
    e = [(k[x], k[y]) for x, y in np.array(edges)[rng.permutation(len(edges))]]
    e += [(a, x) for x in k[rng.permutation(m)]] + [(b, x) for x in k[rng.permutation(m)]] + [(a, b)]
    M = np.full((m + 2, m + 2), 10 ** 6, np.int32)
    for q, (x, y) in enumerate(e):
        M[x, y] = M[y, x] = q + 1
    return M, len(e) + 1


@pytest.mark.parametrize("m", [3, 4, 5, 33, 62, 63, 64, 65, 66])
def test_one_cycle(m):
    _check(*_suspension([(i, (i + 1) % m) for i in range(m)], m, m), f"cycle of {m}")


@pytest.mark.parametrize("p,q", [(2, 2), (3, 3), (8, 8), (9, 9), (9, 10), (20, 4)])
def test_many_cycles(p, q):
    """Complete bipartite links: (p - 1)(q - 1) independent cycles."""
    _check(*_suspension([(i, p + j) for i in range(p) for j in range(q)], p + q, p), f"bipartite {p} {q}")


@pytest.mark.parametrize("parts", [1, 2, 5])
def test_components_and_tails(parts):
    """Cycles of six with a filled triangle on one edge and a path hanging off
    it, and lone vertices."""
    e, m = [], 0
    for _ in range(parts):
        e += [(m + i, m + (i + 1) % 6) for i in range(6)] + [(m, m + 6), (m + 1, m + 6), (m + 2, m + 7), (m + 7, m + 8)]
        m += 9
    _check(*_suspension(e, m + 3, parts), f"{parts} parts")


@pytest.mark.parametrize("copies", [40, 75])
def test_many_triangles(copies):
    """Complexes side by side, each against its own oracle: below and above
    393216 triangles, past which the coboundaries are reduced.  Every tenth
    has random ranks and links with cycles, the others are samples of
    spheres."""
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n0, K0 = 60, 880
    iu = np.triu_indices(n0, 1)
    n = copies * n0
    M = np.full((n, n), 10 ** 8, np.int32)
    small = []
    for c in range(copies):
        g = np.random.default_rng(c)
        if c % 10 == 3:
            order = g.permutation(len(iu[0]))
        else:
            p = g.normal(size=(n0, 3))
            p = np.rint(100 * p / np.linalg.norm(p, axis=1)[:, None]).astype(np.int64)
            order = np.argsort(((p[iu[0]] - p[iu[1]]) ** 2).sum(1), kind="stable")
        rank = np.empty(len(order), np.int64)
        rank[order] = np.arange(len(order))
        m = np.zeros((n0, n0), np.int64)
        m[iu] = rank + 1
        m = m + m.T
        small.append(m.astype(np.int32))
        M[c * n0:(c + 1) * n0, c * n0:(c + 1) * n0] = np.where(m > K0, 10 ** 8, m * copies + c)
    np.fill_diagonal(M, 0)
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), ("sqdist", 10 ** 8, 0), maxdim=3)
    print(f"[gpu] links of {copies} complexes {r.counts}", flush=True)
    e_low, _ = vr.pairs_dim0(r)
    tt = vr.pairs_dim2(r, vr.pairs_dim1(r, e_low)).cpu().numpy()
    tri = (r.tri_key().cpu().numpy() >> 26) & 0x1FFF
    tet = (r.tet_key().cpu().numpy()[:, 1] >> 39) & 0x1FFF
    assert (r.counts[2] > 393216) == (copies == 75)
    r.free()
    for c, m in enumerate(small):
        f = orc.build_matrix(m, ("sqdist", K0 + 1, 0))
        tets = orc.tetra_list(f)
        q_low = orc.reduce_dim2(f, tets, "cohomology", orc.reduce(f, "cohomology").t_low)
        want = np.full(f.T, -1, np.int64)
        want[q_low[q_low >= 0]] = np.nonzero(q_low >= 0)[0]
        at, aq = np.nonzero(tri // n0 == c)[0], np.nonzero(tet // n0 == c)[0]
        assert len(at) == f.T and len(aq) == len(tets)
        assert np.array_equal(tt[at], np.where(want >= 0, aq[want], -1)), c
