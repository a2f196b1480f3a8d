"""Tetrahedra counted and listed from builds up to the edges, which hold no
triangles: the same as from builds with them, whatever kernels take them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K", [(5, 10), (91, 4095), (92, 4186), (150, 11175), (1024, 20000), (1025, 20000)])
def test_without_triangles(n, K):
    import torch

    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] tetra n={n} K={K}", flush=True)
    p = torch.from_numpy(np.random.default_rng(n).integers(-9000, 9000, (n, 3)).astype(np.int16)).to("cuda:0")
    got = []
    for maxdim in (1, 2):
        r = vr.build(p, ("count", K, 1), maxdim=maxdim)
        assert (r.T == 0) == (maxdim == 1)
        off, keys = vr.tetrahedra(r)
        got.append((vr.tetra_counts(r).clone(), off.clone(), keys.clone()))
        r.free()
    assert all(torch.equal(a, b) for a, b in zip(*got))
