"""vr_pairs_dim1 around the limits of the reduction's bits: 2^17 triangles
(16 KB of LDS a wave, or 64) and 2^19 critical triangles (device memory
beyond).  Bit-exact against the oracle; and no jump in the time where the
smaller bits end."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _hub_pairs(pairs, m):
    """Hubs joined to m vertices in random order, then `pairs` edges between
    them, no two closing a triangle of hubs: m - 1 critical triangles each."""
    g = np.random.default_rng(pairs * 10000 + m)
    side = int(np.ceil(np.sqrt(pairs)))
    v = g.permutation(2 * side + m)
    hub, leaf = v[:2 * side], v[2 * side:]
    e = np.array([(h, x) for h in hub for x in leaf])
    e = e[g.permutation(len(e))]
    e = np.concatenate([e, np.array([(a, b) for a in hub[:side] for b in hub[side:]])[:pairs]])
    M = np.full((len(v), len(v)), 10 ** 8, np.int32)
    M[e[:, 0], e[:, 1]] = M[e[:, 1], e[:, 0]] = 1 + np.arange(len(e))
    return M, len(e) + 1


# triangles: 2^17 and 4 more; critical triangles: 2^19 and 128 more
@pytest.mark.parametrize("pairs,m", [(32, 4096), (33, 3972), (128, 4097), (128, 4098)])
def test_limits(pairs, m):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] {pairs} hub edges over {m} vertices", flush=True)
    M, tau = _hub_pairs(pairs, m)
    f = orc.build_matrix(M, ("sqdist", tau, 0))
    p = orc.reduce(f, "cohomology")
    want = np.full(f.K, -1, np.int64)
    want[p.t_low[p.t_low >= 0]] = np.nonzero(p.t_low >= 0)[0]
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), ("sqdist", tau, 0))
    e_low, _ = vr.pairs_dim0(r)
    toe = vr.pairs_dim1(r, e_low).cpu().numpy().astype(np.int64)
    r.free()
    assert np.array_equal(toe, want)


def test_no_jump():
    import torch

    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    took = []
    for pairs in (31, 40):  # 126945 critical triangles, then 163800
        print(f"[gpu] time of {pairs} hub edges", flush=True)
        M, tau = _hub_pairs(pairs, 4096)
        r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), ("sqdist", tau, 0))
        e_low, _ = vr.pairs_dim0(r)
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
    assert took[1] < 3 * took[0]  # the square of the growth is 1.7
