"""Tetrahedra counted and listed by one wave per edge (up to 1024 points, from
4096 edges on, with few triangles an edge) and by four (else): sizes at those
lines and at a wave's width, complete graphs and links of one to a thousand
vertices.  Bit-exact against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(M, K):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    thr = ("sqdist", K + 1, 0)
    f = orc.build_matrix(M, thr)
    want = orc.tetra_list(f)
    print(f"[gpu] tetra n={len(M)} K={f.K} T3={len(want)}", flush=True)
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), thr)
    counts = vr.tetra_counts(r).cpu().numpy()
    off, keys = vr.tetrahedra(r)
    keys = keys.cpu().numpy()
    r.free()
    assert np.array_equal(counts, np.bincount(want[:, 0], minlength=f.K) if len(want) else np.zeros(f.K))
    assert len(keys) == len(want) and int(off[-1]) == len(want)
    if len(want):
        a = want.astype(np.int64)
        assert np.array_equal(keys[:, 0], a[:, 0])
        assert np.array_equal(keys[:, 1], (a[:, 1] << 39) | (a[:, 2] << 26) | (a[:, 3] << 13) | a[:, 4])


def _ranks(n, value):
    """Ranks 1, 2, ... of the pairs in the order of `value`."""
    M = np.zeros((n, n), np.int32)
    iu = np.triu_indices(n, 1)
    order = np.argsort(value, kind="stable")
    M[iu[0][order], iu[1][order]] = np.arange(1, len(order) + 1)
    return M + M.T


@pytest.mark.parametrize("n,degree", [(4, 3), (5, 4), (16, 15), (63, 40), (64, 63), (65, 64), (257, 31), (256, 32), (257, 40),
                                      (257, 90), (257, 130), (1023, 30), (1024, 30), (1025, 30)])
def test_near_points(n, degree):
    rng = np.random.default_rng(n)
    p = rng.integers(-10000, 10001, size=(n, 2)).astype(np.int64)
    iu = np.triu_indices(n, 1)
    q = ((p[iu[0]] - p[iu[1]]) ** 2).sum(1)
    _check(_ranks(n, q), min(len(q), n * degree // 2))


@pytest.mark.parametrize("n", [66, 1024, 1025])
def test_one_large_link(n):
    """A cycle through all vertices but two, with its chords of two and three
    steps, both joined to all, and last to each other: that edge's link holds
    n - 2 vertices."""
    rng = np.random.default_rng(n)
    v = rng.permutation(n)
    a, b, c = v[0], v[1], v[2:]
    e = [(c[k], c[(k + s) % len(c)]) for s in (1, 2, 3) for k in rng.permutation(len(c))]
    e += [(a, x) for x in rng.permutation(c)] + [(b, x) for x in rng.permutation(c)] + [(a, b)]
    M = np.full((n, n), 10 ** 6, np.int32)
    np.fill_diagonal(M, 0)
    for k, (x, y) in enumerate(e):
        M[x, y] = M[y, x] = k + 1
    _check(M, len(e))
