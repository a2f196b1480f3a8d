"""vr_pairs_dim2 from the links at the most triangles that it takes (393216):
every column's bits fill what a launch may have of LDS.  Bit-exact against the
oracle, and without the coboundaries' reduction."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_most_triangles():
    import torch
    from torch.profiler import ProfilerActivity, profile

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 2500
    P = np.random.default_rng(n).integers(-8000, 8000, (n, 2)).astype(np.int64)
    D = ((P[:, None] - P[None]) ** 2).sum(-1)
    tau = int(np.sort(D[np.triu_indices(n, 1)])[49160])
    M, thr = D.astype(np.int32), ("sqdist", tau, 0)
    f = orc.build_matrix(M, thr)
    assert 393184 < f.T <= 393216
    print(f"[gpu] links of {f.T} triangles", flush=True)
    tets = orc.tetra_list(f)
    q_low = orc.reduce_dim2(f, tets, "cohomology", orc.reduce(f, "cohomology").t_low)
    want = np.full(f.T, -1, np.int64)
    want[q_low[q_low >= 0]] = np.nonzero(q_low >= 0)[0]
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), thr, maxdim=3)
    toe = vr.pairs_dim1(r, vr.pairs_dim0(r)[0])
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        tt = vr.pairs_dim2(r, toe).cpu().numpy()
    r.free()
    assert np.array_equal(tt, want)
    ran = {k.key.split("(")[0] for k in p.key_averages()}
    if not any("k_lk_pairs" in k for k in ran):
        pytest.skip("the profiler saw no kernels")
    assert any("k_lk_reduce" in k for k in ran) and not any("k_rd_round" in k for k in ran)
