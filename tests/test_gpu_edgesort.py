"""The edge sort at the lines between its ways of numbering tiles (2048 edges
each): groups of 16 tiles, up to 768 tiles one per work-group, more by
claims.  Against a plain stable sort."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
TILE = 2048


def _check(n, K, distinct):
    import torch

    import paper_1809_04424_amd as vr

    print(f"[gpu] edge sort n={n} K={K} distinct={distinct}", flush=True)
    E = n * (n - 1) // 2
    g = np.random.default_rng(K)
    # exactly K of the pairs lie below K + 1: ranks, or few values below and one above
    q = g.permutation(E) + 1 if distinct else np.where(g.permutation(E) < K, g.integers(1, 300, E), K + 301)
    q = q.astype(np.int32)
    i, j = np.triu_indices(n, 1)
    M = np.zeros((n, n), np.int32)
    M[i, j] = q
    M[j, i] = q
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), ("sqdist", K + 1, 0), maxdim=1)
    order = np.argsort(q, kind="stable")
    order = order[q[order] < K + 1]
    ij, eq = r.edge_ij().cpu().numpy(), r.edge_q().cpu().numpy()
    r.free()
    assert len(order) == K and np.array_equal(eq, q[order])
    assert np.array_equal(ij, np.stack([i[order], j[order]], 1))


@pytest.mark.parametrize("K", [1, TILE, 15 * TILE, 15 * TILE + 1, 16 * TILE, 16 * TILE + 1, 17 * TILE + 5, 33 * TILE])
@pytest.mark.parametrize("distinct", [True, False])
def test_groups(K, distinct):
    _check(400, max(K, 400), distinct)


@pytest.mark.parametrize("tiles", [400, 767, 768, 769, 1025, 2049])
def test_many_tiles(tiles):
    """Of 5.1 million pairs (2498 tiles), so the launch is that for many tiles."""
    _check(3200, tiles * TILE - 3, True)
    _check(3200, tiles * TILE, False)
