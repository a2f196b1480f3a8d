"""Builds of one cloud of up to 128 points (one kernel from the distances to
the kept edges) at the edges of its pairs per thread, passes and staged
coordinates, and just past it.  Bit-exact against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import assert_matches_oracle

pytestmark = pytest.mark.gpu


def _points(n, d, dtype, span, seed):
    g = np.random.default_rng(seed)
    return g.integers(-span, span + 1, (n, d)).astype(dtype)


def _check(orc, data, thr, matrix=False, maxdim=2):
    import torch

    import paper_1809_04424_amd as vr

    x = torch.from_numpy(data).to("cuda:0")
    r = (vr.build_matrix if matrix else vr.build)(x, thr, maxdim=maxdim)
    want = (orc.build_matrix if matrix else orc.build)(data, thr, maxdim=maxdim)
    out = {"counts": r.counts, "edge_ij": r.edge_ij().cpu().numpy().astype(np.int64),
           "edge_q": r.edge_q().cpu().numpy(), "tri": r.tri_key().cpu().numpy()}
    r.free()
    assert_matches_oracle(out, want, check_tri=maxdim >= 2)


@pytest.mark.parametrize("n", [2, 3, 16, 17, 45, 46, 64, 65, 91, 92, 127, 128, 129])
@pytest.mark.parametrize("dtype,span", [("int8", 3), ("int8", 127), ("int16", 30000), ("int32", 15000)])
def test_sizes_and_thresholds(orc, n, dtype, span):
    p = _points(n, 3 if span < 30000 else 1, dtype, span, n)
    print(f"[gpu] small n={n} {dtype} +-{span}", flush=True)
    for thr in (("full", 0, 1), ("fraction", 1, 3), ("count", min(7, n * (n - 1) // 2), 1), ("count", 0, 1),
                ("sqdist", span * span, 0), ("sqdist", 0, 0), ("sqdist", 1 << 40, 0)):
        _check(orc, p, thr)
    _check(orc, p, ("fraction", 1, 2), maxdim=1)


@pytest.mark.parametrize("n,d", [(2, 1000), (64, 31), (64, 32), (64, 33), (64, 128), (64, 131), (128, 32), (128, 33),
                                 (100, 52), (100, 53), (9, 7000)])
def test_coordinates(orc, n, d):
    print(f"[gpu] small n={n} d={d}", flush=True)
    _check(orc, _points(n, d, "int8", 100, d), ("fraction", 1, 2))


@pytest.mark.parametrize("n", [2, 64, 65, 92, 128])
@pytest.mark.parametrize("hi", [1, 2, 255, 256, 257, 65536, 2**24, 2**31 - 1])
def test_matrix_digits(orc, n, hi):
    """Values of 0 to 4 digits, all equal to hardly any equal."""
    M = np.triu(np.random.default_rng(n).integers(0, hi, (n, n)), 1)
    print(f"[gpu] small matrix n={n} below {hi}", flush=True)
    _check(orc, (M + M.T).astype(np.int32), ("fraction", 2, 3), matrix=True)


def test_out_of_range():
    import torch

    import paper_1809_04424_amd as vr

    p = torch.tensor([[0, 0], [65535, 0], [3, 4]], dtype=torch.int32, device="cuda:0")
    r = vr.build(p)
    assert r.edge_q().cpu().tolist() == [25, 65532**2 + 16, 65535**2]
    r.free()
    for bad in ([[0, 0], [65536, 0]], [[0, 0], [65535, 65535]], [[-2**31, 0], [2**31 - 1, 0]]):
        with pytest.raises(vr.VrError) as e:
            vr.build(torch.tensor(bad, dtype=torch.int32, device="cuda:0"))
        assert e.value.code == vr.VR_ERANGE
    M = torch.tensor([[0, -1, 2], [-1, 0, 3], [2, 3, 0]], dtype=torch.int32, device="cuda:0")
    with pytest.raises(vr.VrError) as e:
        vr.build_matrix(M)
    assert e.value.code == vr.VR_ERANGE
