"""The triangle write's default of one or two work-groups a vertex, at the line
between them and past the points where the line stays: the same keys as with
either pinned."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2100, 4100, 6000])
@pytest.mark.parametrize("off", [-1, 0])
def test_line(n, off):
    import torch

    import paper_1809_04424_amd as vr

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    K = (n * (250 + n // 32) + 1) // 2 + off
    print(f"[gpu] {n} points, {K} edges", flush=True)
    P = torch.from_numpy(np.random.default_rng(n).integers(-4000, 4000, (n, 3)).astype(np.int32)).to("cuda:0")
    thr = ("count", K, 1)
    first = vr.build(P, thr)
    keys = first.tri_key()
    for parts in (1, 2):
        vr.set_schedule(P, thr, (512, 1, 4, 512, parts, 8))
        r = vr.build(P, thr)
        assert torch.equal(r.tri_key(), keys)
        r.free()
    first.free()
