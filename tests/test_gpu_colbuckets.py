"""vr_column_order's ways of ranking a window (counting, buckets of values, 32-bit
keys, 64-bit keys) at the lines between them.
Bit-exact against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
WIN = 4096


def _check(orc, lens, v, label):
    import torch

    import paper_1809_04424_amd as vr

    print(f"[gpu] column order {label}", flush=True)
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    v = np.ascontiguousarray(v, np.int32)
    assert len(v) == cp[-1]
    z = vr.column_order(torch.from_numpy(cp).to("cuda:0"), torch.from_numpy(v).to("cuda:0")).cpu().numpy()
    assert np.array_equal(z, orc.column_order(cp, v))


@pytest.mark.parametrize("segments", [2, 128, 255, 256, 257, 258, 1500])
@pytest.mark.parametrize("hi", [2, 40, 2**17, 2**31 - 1])
def test_segments_of_a_window(orc, segments, hi):
    """One segment of 257 or more and short ones around it, twice over."""
    g = np.random.default_rng(segments)
    lens = np.ones(segments, np.int64)
    lens[segments // 2] = max(257, 2500 - segments)
    lens = np.tile(lens, 2)
    _check(orc, lens, g.integers(0, hi, lens.sum()), f"{segments} segments below {hi}")


@pytest.mark.parametrize("same", [1, 23, 24, 25, 26, 300, 1999])
@pytest.mark.parametrize("spread", [2**12, 2**20, 2**32])
def test_equal_values(orc, same, spread):
    """Equal values among spread ones, around the longest bucket allowed; the
    spread values take 12 bits (32-bit keys), 20 and 32 (64-bit keys)."""
    g = np.random.default_rng(same)
    lens = [1999, 1999, 700]
    v = g.integers(-(spread // 2), spread // 2, sum(lens))
    for lo, n in ((0, 1999), (1999, 1999), (3998, 700)):
        at = lo + g.choice(n, min(same, n), replace=False)
        v[at] = spread // 4
    _check(orc, lens, v, f"{same} equal, spread {spread}")


@pytest.mark.parametrize("bits", [17, 18, 19, 31])
@pytest.mark.parametrize("segments", [1, 2, 3, 4])
def test_bits_of_the_keys(orc, bits, segments):
    """Clustered values (no buckets) whose keys just fit 32 bits, or do not."""
    g = np.random.default_rng(bits)
    lens = np.full(segments, WIN // segments)
    v = g.integers(0, 30, lens.sum())
    v[np.cumsum(lens) - 1] = 2**bits - 1
    _check(orc, lens, v, f"{bits} bits, {segments} segments")


@pytest.mark.parametrize("nnz", [257, 300, 4095, 4096, 4097, 8191, 12289])
def test_extremes(orc, nnz):
    g = np.random.default_rng(nnz)
    v = g.integers(-2**31, 2**31, nnz)
    v[g.choice(nnz, 20, replace=False)] = np.repeat([-2**31, 2**31 - 1], 10)
    _check(orc, [nnz], v, f"extremes {nnz}")


@pytest.mark.parametrize("length", [1, 8, 23, 24, 25, 26, 255, 256, 257])
@pytest.mark.parametrize("rest", [0, 3, 254, 255, 256, 900])
def test_counted_and_not(orc, length, rest):
    """The longest segment around the two counting limits, with up to and more
    than 256 segments in the window; few values, so that many are equal."""
    g = np.random.default_rng(length + rest)
    lens = np.concatenate([g.integers(0, min(length, 4) + 1, rest), [length], g.integers(0, 3, rest // 2)])
    v = g.integers(-3, 4, lens.sum()) if rest % 2 else g.integers(-2**31, 2**31, lens.sum())
    _check(orc, lens, v, f"longest {length}, {len(lens)} columns")
