"""Clouds far from the origin: only the differences of their coordinates
count, whatever the number of points, the kernel that takes the distances (a
build timed stage by stage has its own) and the coordinates staged at a time.
Bit-exact against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import assert_matches_oracle, item_host

pytestmark = pytest.mark.gpu
FAR = [100000, -100000, 2**31 - 201, -(2**31)]


def _ways(p, thr):
    """One cloud's result from a plain build, a timed one and a captured one."""
    import torch

    import paper_1809_04424_amd as vr

    x = torch.from_numpy(p).to("cuda:0")
    for way, kw in (("plain", {}), ("timed", {"timing": True}), ("captured", {"graph": True})):
        r = vr.build(x, thr, **kw)
        yield way, item_host(r)
        r.free()


@pytest.mark.parametrize("n", [65, 100, 128, 129, 130, 200])
@pytest.mark.parametrize("d", [3, 9, 70])
@pytest.mark.parametrize("far", FAR)
def test_translated(orc, n, d, far):
    print(f"[gpu] translated n={n} d={d} by {far}", flush=True)
    p = (np.random.default_rng(n * d).integers(0, 201, (n, d)) + far).astype(np.int32)
    want = orc.build(p, ("fraction", 1, 3))
    for way, out in _ways(p, ("fraction", 1, 3)):
        print(f"[gpu] {way}", flush=True)
        assert_matches_oracle(out, want)


@pytest.mark.parametrize("n", [65, 129, 130])
@pytest.mark.parametrize("at", [0, -1])
def test_too_far_apart(n, at):
    """One point 65536 away from the others is refused every way."""
    import torch

    import paper_1809_04424_amd as vr

    p = torch.full((n, 3), 100000, dtype=torch.int32)
    p[at, 1] += 65536
    x = p.to("cuda:0")
    thr = ("fraction", 1, 3)
    for call in (lambda: vr.build(x, thr), lambda: vr.build(x, thr, timing=True),
                 lambda: vr.build(x, thr, graph=True)):
        with pytest.raises(vr.VrError) as e:
            call()
        assert e.value.code == vr.VR_ERANGE
