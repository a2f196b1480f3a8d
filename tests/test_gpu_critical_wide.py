"""vr_pairs_dim1 on edges whose common neighbours fall into many components,
or into few that take long to search: on both sides of the vertices that a
wave holds and of the length at which the search is left to a pass over the
older edges.  Bit-exact against the oracle; and such an edge's time grows with
its neighbours and not with their square."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _hubs(m, shape, hubs, before, seed):
    """`before` edges of a path of its own, then edges among m vertices, then
    those to each of the hubs in random order, then the hubs' edges with one
    another: each of the m is a common neighbour of every pair of hubs.  The
    earliest spokes of the first two hubs lead to one vertex in the middle, so
    that the search does not begin at the first component."""
    g = np.random.default_rng(seed)
    n = m + hubs + before + 1
    v = g.permutation(n)
    x, h, path = v[:m], v[m:m + hubs], v[m + hubs:]
    e = [(path[i], path[i + 1]) for i in range(before)]
    x = np.sort(x)  # components in the order of their vertices, unless shuffled below
    if shape == "pairs":
        e += [(x[i], x[i + 1]) for i in range(0, m - 1, 2)]
    elif shape == "halves":
        e += [(x[i], x[i + 2]) for i in range(m - 2)]
    elif shape == "quarter and lone":
        y = g.permutation(x)
        e += [(y[i], y[i + 1]) for i in range(m // 4)]
    elif shape == "path":
        y = g.permutation(x)
        e += [(y[i], y[i + 1]) for i in range(m - 1)]
    mid = x[m // 2]
    e += [(h[0], mid), (h[1], mid)]
    spokes = [(a, b) for a in h for b in x if not (b == mid and a in (h[0], h[1]))]
    e += [spokes[i] for i in g.permutation(len(spokes))]
    e += [(h[i], h[j]) for i in range(hubs) for j in range(i)]
    M = np.full((n, n), 10 ** 7, np.int32)
    e = np.array(e)
    M[e[:, 0], e[:, 1]] = M[e[:, 1], e[:, 0]] = 1 + np.arange(len(e))
    return M, len(e) + 1


def _resident(M, tau):
    import torch

    import paper_1809_04424_amd as vr

    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), ("sqdist", tau, 0))
    return r, vr.pairs_dim0(r)[0]


@pytest.mark.parametrize("shape", ["lone", "pairs", "halves", "quarter and lone", "path"])
@pytest.mark.parametrize("m,hubs,before", [(62, 2, 0), (64, 2, 0), (65, 2, 0), (66, 2, 0), (66, 2, 2000), (130, 3, 0),
                                           (384, 2, 0), (390, 2, 0), (512, 3, 0), (513, 3, 0), (1100, 2, 0), (3000, 2, 0)])
def test_links(shape, m, hubs, before):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] {hubs} hubs over {m} vertices, {shape}, after {before} edges", flush=True)
    M, tau = _hubs(m, shape, hubs, before, m + before)
    f = orc.build_matrix(M, ("sqdist", tau, 0))
    p = orc.reduce(f, "cohomology")
    want = np.full(f.K, -1, np.int64)
    want[p.t_low[p.t_low >= 0]] = np.nonzero(p.t_low >= 0)[0]
    r, e_low = _resident(M, tau)
    for _ in range(2):  # the second call finds the first one's scratch
        toe = vr.pairs_dim1(r, e_low).cpu().numpy().astype(np.int64)
        assert np.array_equal(toe, want)
    r.free()


def test_time_grows_with_the_neighbours():
    import torch

    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    took = []
    for m in (2000, 8000):
        print(f"[gpu] an edge with {m} common neighbours", flush=True)
        r, e_low = _resident(*_hubs(m, "lone", 2, 0, m))
        best = 1e9
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            vr.pairs_dim1(r, e_low)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        r.free()
        took.append(best)
    print(f"[gpu] {took[0] * 1e6:.0f} us, then {took[1] * 1e6:.0f}", flush=True)
    assert took[1] < 8 * took[0]  # four times the neighbours; the square would be 16
