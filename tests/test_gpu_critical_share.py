"""vr_pairs_dim1 around the critical triangles that one share of the edges may
find (2^22 in 16 shares, edges to a share 16 at a time): below, they are
reduced; past it the edge columns themselves are (in scratch of over 1 GiB).
Bit-exact against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hub_edges,past", [(131, False), (132, True)])
def test_one_share(hub_edges, past):
    """23 hubs joined to 2000 vertices in random order (46000 edges: whole
    sixteens), then edges between the first 12 hubs and the others, each with
    those 2000 as common neighbours, no two joined: 1999 critical triangles
    each, all in one share, for 240 edges of a path come after every 16."""
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] one share, {hub_edges} hub edges", flush=True)
    g = np.random.default_rng(hub_edges)
    gaps = (hub_edges + 15) // 16
    n = 23 + 2000 + 240 * gaps + 1
    v = g.permutation(n)
    hub, leaf, path = v[:23], v[23:2023], v[2023:]
    first = np.array([(h, x) for h in hub for x in leaf])
    first = first[g.permutation(len(first))]
    pairs = np.array([(a, b) for a in hub[:12] for b in hub[12:]])[:hub_edges]
    e = [first]
    for k in range(gaps):
        e += [pairs[16 * k:16 * k + 16], np.stack([path[240 * k:240 * k + 240], path[240 * k + 1:240 * k + 241]], 1)]
    e = np.concatenate(e)
    M = np.full((n, n), 10 ** 7, np.int32)
    M[e[:, 0], e[:, 1]] = M[e[:, 1], e[:, 0]] = 1 + np.arange(len(e))
    thr = ("sqdist", len(e) + 1, 0)
    f = orc.build_matrix(M, thr)
    p = orc.reduce(f, "cohomology")
    want = np.full(f.K, -1, np.int64)
    want[p.t_low[p.t_low >= 0]] = np.nonzero(p.t_low >= 0)[0]
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), thr)
    e_low, _ = vr.pairs_dim0(r)
    torch.cuda.synchronize()
    vr.trim()
    toe = vr.pairs_dim1(r, e_low).cpu().numpy().astype(np.int64)
    held = vr.trim()
    r.free()
    assert np.array_equal(toe, want)
    assert (held > 1 << 30) == past, held
