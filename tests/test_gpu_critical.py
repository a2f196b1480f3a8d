"""vr_pairs_dim1 on the critical cells, where its pieces end: the common
neighbours of one edge (64 to a piece, 512 in registers, more from memory) and
the critical triangles a column has bits for (2^17 in LDS, more in memory).
Bit-exact against the oracle's reduction."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def hub_matrix(m, joined):
    """Vertices a = 0, b = 1, c, d and k_0 .. k_{m-1} (shuffled).  The path
    a-c-d-b is oldest, then the edges a k_i, then b k_i, each of which closes a
    cycle, and last a b, which k_0 .. k_{m-1} fill: k_0's cycle lies in the
    boundary of m - 1 critical triangles.  With `joined`, k_i and k_{i+1} are
    joined before that for even i, so that half the components are pairs."""
    rng = np.random.default_rng(m)
    n = m + 4
    M = np.full((n, n), 10 ** 6, np.int64)
    k = 4 + rng.permutation(m)
    edges = [(0, 2), (2, 3), (1, 3)] + [(0, x) for x in k] + [(1, x) for x in k]
    if joined:
        edges += [(k[i], k[i + 1]) for i in range(0, m - 1, 2)]
    edges.append((0, 1))
    for q, (x, y) in enumerate(edges):
        M[x, y] = M[y, x] = q + 1
    return M.astype(np.int32), len(edges) + 1


@pytest.mark.parametrize("joined", [False, True])
@pytest.mark.parametrize("m", [1, 2, 64, 65, 511, 512, 513, 2049])
def test_hub_edge(m, joined):
    print(f"[gpu] hub edge m={m} joined={joined}", flush=True)
    _check(*hub_matrix(m, joined))


@pytest.mark.parametrize("h,m", [(3, 100), (93, 1410), (94, 1410)])
def test_hub_pairs(h, m):
    """h pairs of hubs, every hub joined to m vertices in random order, then
    each pair's hubs to each other: h (m - 1) critical triangles (2^17 lies
    between the last two) and (2 h - 1)(m - 1) critical edges."""
    print(f"[gpu] hub pairs h={h} m={m}", flush=True)
    rng = np.random.default_rng(h)
    n = 2 * h + m
    v = rng.permutation(n)
    edges = np.array([(x, y) for x in v[:2 * h] for y in v[2 * h:]])
    edges = np.concatenate([edges[rng.permutation(len(edges))], v[:2 * h].reshape(h, 2)])
    M = np.full((n, n), 10 ** 7, np.int32)
    M[edges[:, 0], edges[:, 1]] = M[edges[:, 1], edges[:, 0]] = 1 + np.arange(len(edges))
    _check(M, len(edges) + 1)


@pytest.mark.parametrize("n", [66, 200])
def test_random_ranks(n):
    """Edges in random order: common neighbours stay unjoined far into the
    filtration, and the critical edges lie in many boundaries."""
    print(f"[gpu] random ranks n={n}", flush=True)
    rng = np.random.default_rng(n)
    M = np.zeros((n, n), np.int64)
    iu = np.triu_indices(n, 1)
    M[iu] = 1 + rng.permutation(len(iu[0]))
    _check((M + M.T).astype(np.int32), int(len(iu[0]) * 0.28))


def _check(M, tau):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f = orc.build_matrix(M, ("sqdist", tau, 0))
    p = orc.reduce(f, "cohomology")
    want = np.full(f.K, -1, np.int64)
    for t in np.nonzero(p.t_low >= 0)[0]:
        want[p.t_low[t]] = t
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), ("sqdist", tau, 0))
    e_low, _ = vr.pairs_dim0(r)
    toe = vr.pairs_dim1(r, e_low)
    assert np.array_equal(e_low.cpu().numpy(), p.e_low)
    assert np.array_equal(toe.cpu().numpy().astype(np.int64), want)
    r.free()
