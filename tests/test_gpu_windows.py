"""Buckets sorted in LDS: windows whose keys lie evenly, in runs of equal keys, in
clusters with a gap between them (of spans below and beyond 51 bits, where keys
closer than the dropped bits occur or not), at sizes around the workgroup, the
slot and the largest window.  Exact against a stable sort."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tqp():
    import paper_2209_04579_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def keys_of(kind, n, rng):
    if kind == "even":
        return rng.integers(0, 1 << 40, n)
    if kind == "values":                       # a bin per value, mostly crowded
        return rng.integers(0, 300, n)
    if kind == "exponential":                  # crowded bins at one end
        return np.exp(rng.uniform(0, 33, n)).astype(np.int64)
    far = {"gap50": 50, "gap52": 52, "gap61": 61}[kind.split("-")[0]]
    step = {"dense": 1, "loose": 1 << 13}[kind.split("-")[1]]
    near = rng.integers(0, 3 * n, n) * step
    return np.where(rng.random(n) < 0.3, near, near + (1 << far))


@pytest.mark.parametrize("n", [2, 8, 9, 1023, 5119, 5121, 8191, 8192, 8193, 60_001])
@pytest.mark.parametrize("kind", ["even", "values", "exponential", "gap50-dense", "gap52-dense", "gap52-loose",
                                  "gap61-dense", "gap61-loose"])
def test_window_forms(tqp, kind, n):
    k = keys_of(kind, n, np.random.default_rng(n))
    k = k.astype(np.int64) - (1 << 39)
    k[0], k[-1] = k.max(), k.min()             # the ends of the span in the wrong order
    key = torch.from_numpy(k).cuda()
    bits = 1 if n < 10_000 else 4
    got, rows, _ = tqp.partition_sort(key, mode=tqp.PART_RADIX, bucket_bits=bits)
    want = np.argsort(k, kind="stable")
    assert np.array_equal(rows.cpu().numpy(), want)
    assert np.array_equal(got.cpu().numpy(), k[want])
    if kind in ("even", "values", "exponential"):
        k32 = (k >> 9).astype(np.int32)
        got, rows, _ = tqp.partition_sort(torch.from_numpy(k32).cuda(), mode=tqp.PART_RADIX, bucket_bits=bits)
        want = np.argsort(k32, kind="stable")
        assert np.array_equal(rows.cpu().numpy(), want)
        assert np.array_equal(got.cpu().numpy(), k32[want])
