"""Candidate lists at the edges of the enumeration's pieces (64 entries), of
the pieces kept in registers (256 or 512) and of the staged hits, for the count
and both writers.  Bit-exact against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import assert_matches_oracle

pytestmark = pytest.mark.gpu
FAR = 1 << 24


def _complete(n):
    """All edges in a random order: the lists reach n - 1 entries."""
    return np.random.default_rng(n).integers(1, 1 << 20, (n, n)).astype(np.int32)


def _hubs(n, hubs=7):
    """A path and hubs adjacent to every vertex; the edges between hubs come
    last: their lists have all n - 1 entries, nearly all hits."""
    M = np.full((n, n), FAR, np.int32)
    g = np.random.default_rng(n)
    M[np.arange(n - 1), np.arange(1, n)] = g.integers(1, 1 << 10, n - 1)
    h = g.choice(n, hubs, replace=False)
    M[h, :] = g.integers(1, 1 << 10, (hubs, n))
    M[:, h] = M[h, :].T
    M[np.ix_(h, h)] = 1 << 11
    return M


@pytest.mark.parametrize("shape,n", [("complete", n) for n in (3, 4, 17, 65, 66, 129, 257, 258, 273)]
                         + [("hubs", n) for n in (320, 385, 513, 514, 515, 577, 641, 769, 1025, 1100)])
def test_lists(orc, shape, n):
    import torch

    import paper_1809_04424_amd as vr

    M = np.triu((_complete if shape == "complete" else _hubs)(n), 1)
    M = M + M.T
    thr = ("sqdist", FAR, 0)
    want = orc.build_matrix(M, thr)
    d = torch.from_numpy(M).to("cuda:0")
    for sched in (None, (128, 1, 2, 128, 1, 4), (256, 2, 8, 256, 0, 4), (512, 1, 4, 128, 0, 8), (256, 8, 4, 512, 8, 8)):
        print(f"[gpu] lists {shape} n={n} {sched}", flush=True)
        if sched:
            vr.set_schedule(d, thr, sched, matrix=True)
        r = vr.build_matrix(d, thr)
        out = {"counts": r.counts, "edge_ij": r.edge_ij().cpu().numpy().astype(np.int64),
               "edge_q": r.edge_q().cpu().numpy(), "tri": r.tri_key().cpu().numpy()}
        r.free()
        assert_matches_oracle(out, want)


@pytest.mark.parametrize("n,K", [(90, 900), (640, 180000), (2100, 30000), (2100, 700000)])
def test_entries_left_from_a_build_of_the_same_tag(n, K):
    """Row entries that an earlier build left and that carry the same tag (one
    build in 255) are candidates for a star and fail the look-up."""
    import torch

    import paper_1809_04424_amd as vr

    g = np.random.default_rng(n)
    a, b, small = (torch.from_numpy(g.integers(-90, 91, (m, 3)).astype(np.int8)).to("cuda:0") for m in (n, n, 9))

    def out(p):
        r = vr.build(p, ("count", K, 1))
        o = [x.cpu().numpy() for x in (r.edge_ij(), r.edge_q(), r.tri_key())]
        r.free()
        return o

    want = out(b)
    for between in (253, 254, 255):
        print(f"[gpu] same tag n={n} after {between}", flush=True)
        out(a)
        for _ in range(between):
            vr.build(small).free()
        assert all(np.array_equal(x, y) for x, y in zip(out(b), want))
