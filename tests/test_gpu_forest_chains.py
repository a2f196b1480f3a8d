"""vr_pairs_dim0 on chains whose edges come from the far end: each joins a
vertex to a component with a larger root, so a round settles one edge a chain
and one wave takes the rest.  One chain to a hundred, alone or after edges that
join at once, at the edges of a wave's 64 and of the rounds that count.
Bit-exact against the oracle; and no chain takes the time of a thread that goes
edge by edge."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _chains(n, chains, front):
    """Vertices 0 .. n - 1 in `chains` runs, each run's edges from its far end,
    in turn; before them `front` edges between further vertices, two by two."""
    runs = np.array_split(np.arange(n), chains)
    e = [(r[k], r[k + 1]) for k in range(max(map(len, runs)) - 2, -1, -1) for r in runs if k + 1 < len(r)]
    e = [(n + 2 * i, n + 2 * i + 1) for i in range(front)] + e
    m = n + 2 * front
    M = np.full((m, m), 10 ** 8, np.int32)
    x, y = np.array(e).T
    M[x, y] = M[y, x] = 1 + np.arange(len(e))
    return M, ("sqdist", len(e) + 1, 0)


@pytest.mark.parametrize("n,chains,front", [(41, 1, 0), (42, 1, 0), (64, 1, 0), (65, 1, 0), (66, 1, 7), (130, 2, 0),
                                            (1200, 13, 0), (1200, 14, 0), (1200, 100, 0), (1000, 1, 900), (3000, 1, 60)])
def test_chains(n, chains, front):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    print(f"[gpu] chains n={n} chains={chains} front={front}", flush=True)
    M, thr = _chains(n, chains, front)
    want = orc.reduce(orc.build_matrix(M, thr), "cohomology").e_low
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), thr, maxdim=1)
    e_low, death = (x.cpu().numpy().astype(np.int64) for x in vr.pairs_dim0(r))
    r.free()
    back = np.full(len(M), -1, np.int64)
    back[want[want >= 0]] = np.nonzero(want >= 0)[0]
    assert np.array_equal(e_low, want) and np.array_equal(death, back)


def test_time_of_a_chain():
    """About 4 times a shuffled path's; edge by edge it took 14 times."""
    import torch

    import paper_1809_04424_amd as vr

    def us(M, thr):
        r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), thr, maxdim=1)
        best = 1e9
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            vr.pairs_dim0(r)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3)
        r.free()
        return best

    n = 4200
    M, thr = _chains(n, 1, 0)
    p = np.random.default_rng(1).permutation(n)
    chain, shuffled = us(M, thr), us(M[p][:, p], thr)
    print(f"[gpu] chain {chain:.0f} us, shuffled {shuffled:.0f} us", flush=True)
    assert chain < 10 * shuffled
