"""vr_pairs_dim0's spanning forest at the edges of its stretches (2n edges,
then three times as many as came before) and batches (2048 marked edges), and on
chains that join one edge a round.  Bit-exact against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(M, tau):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f = orc.build_matrix(M, ("sqdist", tau, 0))
    want = orc.reduce(f, "cohomology").e_low
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), ("sqdist", tau, 0))
    e_low, death = (x.cpu().numpy().astype(np.int64) for x in vr.pairs_dim0(r))
    r.free()
    assert np.array_equal(e_low, want)
    back = np.full(len(M), -1, np.int64)
    back[want[want >= 0]] = np.nonzero(want >= 0)[0]
    assert np.array_equal(death, back)


def _matrix(n, edges):
    M = np.full((n, n), 10 ** 8, np.int32)
    x, y = edges[:, 0], edges[:, 1]
    M[x, y] = M[y, x] = 1 + np.arange(len(edges))
    return M, len(edges) + 1


@pytest.mark.parametrize("order", ["forward", "backward", "shuffled"])
@pytest.mark.parametrize("n", [2, 3, 64, 1025, 2049, 2050, 4200])
def test_path(n, order):
    """A path whose edges come in order (each joins the growing component: one
    a round), from the other end, or shuffled."""
    print(f"[gpu] forest path n={n} {order}", flush=True)
    i = np.arange(n - 1)
    i = i if order == "forward" else i[::-1] if order == "backward" else np.random.default_rng(n).permutation(n - 1)
    _check(*_matrix(n, np.stack([i, i + 1], 1)))


@pytest.mark.parametrize("n", [70, 700])
@pytest.mark.parametrize("k", ["2n-1", "2n", "2n+1", "4n", "4n+1", "8n+63"])
def test_random_edges(n, k):
    """The first edges of a random order, in two halves that no edge joins."""
    print(f"[gpu] forest n={n} K={k}", flush=True)
    rng = np.random.default_rng(n)
    iu = np.stack(np.triu_indices(n, 1), 1)
    iu = iu[(iu[:, 0] % 2) == (iu[:, 1] % 2)]
    edges = iu[rng.permutation(len(iu))][:eval(k.replace("n", "*n"))]
    _check(*_matrix(n, edges))
