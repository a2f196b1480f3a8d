"""vr_column_order where values crowd: seen in the first quarter of a window or
only later, at the count that ends the buckets, and sorted by 32-bit and
64-bit keys in windows of one to many segments.  Bit-exact against the oracle;
and crowded values take little longer than spread ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
WIN = 4096


def _order(cp, v):
    import torch

    import paper_1809_04424_amd as vr

    cp, v = torch.from_numpy(cp).to("cuda:0"), torch.from_numpy(v).to("cuda:0")
    return lambda: vr.column_order(cp, v)


def _check(orc, lens, v, label):
    print(f"[gpu] column order {label}", flush=True)
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    v = np.ascontiguousarray(np.clip(v, -2**31, 2**31 - 1), np.int32)
    assert np.array_equal(_order(cp, v)().cpu().numpy(), orc.column_order(cp, v))


def _crowded(name, u):
    g = np.random.default_rng(1)
    return {"twelfth powers": u ** 12 * 2**31, "cubes": u ** 3 * 2**32 - 2**31, "lognormal": np.exp(4 * g.standard_normal(len(u))),
            "both ends": np.where(u < 0.5, -2.0**31 + 10 * u, 2.0**31 - 1 - 10 * u), "few": np.floor(u * 5),
            "one far": np.where(u < 1e-3, 2.0**31 - 1, u * 40)}[name]


@pytest.mark.parametrize("kind", ["twelfth powers", "cubes", "lognormal", "both ends", "few", "one far"])
@pytest.mark.parametrize("lens", [[4096], [4095], [4097, 25], [9000], [1999, 1999, 1999], [300] * 40, [25] * 400, [16] * 600,
                                  [2000, 1, 0, 2] * 5], ids=str)
def test_crowded(orc, kind, lens):
    u = np.random.default_rng(len(lens)).random(sum(lens))
    _check(orc, lens, _crowded(kind, u), f"{kind} {lens[:4]} x {len(lens)}")


@pytest.mark.parametrize("same", [23, 24, 25, 26, 100])
@pytest.mark.parametrize("first", [0, 1000, 1024, 3000])
def test_place_of_the_crowd(orc, same, first):
    """Equal values from position `first` on among spread ones."""
    v = np.random.default_rng(same).integers(-2**31, 2**31, 2 * WIN + 5)
    for w in (0, WIN):
        v[w + first:w + first + same] = 12345
    _check(orc, [len(v)], v, f"{same} equal from {first}")


def test_time_of_crowded_values():
    """1.5 times the spread values'; twice before the sort was made up to it."""
    import torch

    u = np.random.default_rng(5).random(2000 * 1999)
    cp = np.arange(2001, dtype=np.int64) * 1999
    us = []
    for x in (u * 2**20, np.minimum(_crowded("lognormal", u), 2e9)):
        f = _order(cp, x.astype(np.int32))
        best = 1e9
        for _ in range(30):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            f()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3)
        us.append(best)
    print(f"[gpu] spread {us[0]:.0f} us, crowded {us[1]:.0f}", flush=True)
    assert us[1] < 1.75 * us[0], us
