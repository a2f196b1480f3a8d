"""vr_pairs_dim2 where many columns of critical tetrahedra are left to reduce:
grids, whose equal distances leave hundreds, in the grid's order and in a
random one.  Bit-exact against the oracle; and reducing the columns takes less
of the time than finding them, for few of them meet."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _grid(side, shuffled):
    g = np.stack(np.meshgrid(*[np.arange(s) for s in side], indexing="ij"), -1).reshape(-1, len(side)).astype(np.int64)
    if shuffled:
        g = g[np.random.default_rng(len(g)).permutation(len(g))]
    return ((g[:, None] - g[None]) ** 2).sum(-1).astype(np.int32)


@pytest.mark.parametrize("side,tau", [((3, 3, 3), 13), ((4, 4, 4), 7), ((6, 5, 4), 7), ((7, 7, 2), 6), ((12, 12), 9), ((3, 3, 3, 2), 6)])
@pytest.mark.parametrize("shuffled", [False, True])
def test_grids(side, tau, shuffled):
    import torch

    import oracle as orc
    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] grid {side} shuffled={shuffled}", flush=True)
    M, thr = _grid(side, shuffled), ("sqdist", tau, 0)
    f = orc.build_matrix(M, thr)
    tets = orc.tetra_list(f)
    q_low = orc.reduce_dim2(f, tets, "cohomology", orc.reduce(f, "cohomology").t_low)
    want = np.full(f.T, -1, np.int64)
    want[q_low[q_low >= 0]] = np.nonzero(q_low >= 0)[0]
    r = vr.build_matrix(torch.from_numpy(M).to("cuda:0"), thr, maxdim=3)
    e_low, _ = vr.pairs_dim0(r)
    tt = vr.pairs_dim2(r, vr.pairs_dim1(r, e_low)).cpu().numpy()
    r.free()
    assert np.array_equal(tt, want)


def test_share_of_the_time():
    import torch
    from torch.profiler import ProfilerActivity, profile

    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[gpu] grid 8 8 8", flush=True)
    r = vr.build_matrix(torch.from_numpy(_grid((8, 8, 8), False)).to("cuda:0"), ("sqdist", 7, 0), maxdim=3)
    e_low, _ = vr.pairs_dim0(r)
    toe = vr.pairs_dim1(r, e_low)
    vr.pairs_dim2(r, toe)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        for _ in range(5):
            vr.pairs_dim2(r, toe)
        torch.cuda.synchronize()
    r.free()
    took = {k.key.split("(")[0]: k.device_time_total for k in p.key_averages()}
    reduce, expand = (sum(v for k, v in took.items() if name in k) for name in ("k_lk_reduce", "k_lk_expand"))
    if expand == 0:
        pytest.skip("the profiler saw no kernels")
    print(f"[gpu] found in {expand / 5:.0f} us, reduced in {reduce / 5:.0f}", flush=True)
    assert reduce < expand
