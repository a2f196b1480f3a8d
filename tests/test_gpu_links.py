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
