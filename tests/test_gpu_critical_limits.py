"""vr_pairs_dim1 at and past a limit of the reduction on the critical cells:
one critical triangle whose boundary takes a thousand replacements, one by
one, and as many critical edges.  Past it the edge columns themselves are
reduced (in scratch of over 1 GiB).  Bit-exact against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def ladder(m):
    """Vertices v_0 .. v_m and s_0 .. s_m (shuffled).  Oldest: the path of the
    s and the rungs v_i s_i, a tree.  Then the edges v_i v_{i+1}, each of which
    closes a cycle of four and has no common neighbour: critical.  Then the
    fan v_0 v_2, v_0 v_3, ..., each with v_0 v_{k-1} and v_{k-1} v_k as its
    only triangle, and s_0 s_m.  Last v_m s_0, whose common neighbours v_0
    and s_m are not joined: two components."""
    p = np.random.default_rng(m).permutation(2 * m + 2)
    v, s = p[:m + 1], p[m + 1:]
    edges = [(s[i], s[i + 1]) for i in range(m)] + [(v[i], s[i]) for i in range(m + 1)]
    edges += [(v[i], v[i + 1]) for i in range(m)] + [(v[0], v[k]) for k in range(2, m + 1)]
    edges += [(s[0], s[m]), (v[m], s[0])]
    M = np.full((2 * m + 2, 2 * m + 2), 10 ** 6, np.int32)
    for q, (x, y) in enumerate(edges):
        M[x, y] = M[y, x] = q + 1
    return M, len(edges) + 1


@pytest.mark.parametrize("m,past", [(3, False), (1000, False), (1100, True)])
def test_long_replacement(m, past):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] ladder m={m}", flush=True)
    M, tau = ladder(m)
    f = orc.build_matrix(M, ("sqdist", tau, 0))
    p = orc.reduce(f, "cohomology")
    want = np.full(f.K, -1, np.int64)
    for t in np.nonzero(p.t_low >= 0)[0]:
        want[p.t_low[t]] = t
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), ("sqdist", tau, 0))
    e_low, _ = vr.pairs_dim0(r)
    torch.cuda.synchronize()
    vr.trim()
    toe = vr.pairs_dim1(r, e_low).cpu().numpy().astype(np.int64)
    held = vr.trim()
    r.free()
    assert np.array_equal(toe, want)
    assert (held > 1 << 30) == past, held
