"""Buckets sorted in LDS whose keys repeat: a window is merged without a count of its bins
from eight equal neighbours (of one thread, 1024 rows apart) on, else counted.  Runs of
equal keys of every length around that, equal neighbours planted one by one, and windows
of both kinds beside one another.  Exact against a stable sort."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(k):
    import paper_2209_04579_amd as tqp
    for dt in (np.int64, np.int32):
        c = k.astype(dt)
        got, rows, _ = tqp.partition_sort(torch.from_numpy(c).cuda(), mode=tqp.PART_RADIX, bucket_bits=4)
        want = np.argsort(c, kind="stable")
        assert np.array_equal(rows.cpu().numpy(), want)
        assert np.array_equal(got.cpu().numpy(), c[want])


@pytest.mark.parametrize("n", [4000, 50_000])
@pytest.mark.parametrize("run", [2, 6, 8, 12, 16, 17, 30, 300, 4000])
def test_runs(run, n):
    k = np.random.default_rng(run).integers(0, n // run, n) * (3000 if run > 2 else 1) - 70_000
    check(k)


@pytest.mark.parametrize("pairs", [0, 1, 7, 8, 9, 40])
@pytest.mark.parametrize("n", [1025, 3000, 8000])
def test_planted_pairs(pairs, n):
    rng = np.random.default_rng(pairs + n)
    k = rng.permutation(n) * 7
    pairs = min(pairs, n - 1024)
    k[1024:1024 + pairs] = k[:pairs]
    check(k)


def test_both_kinds():
    rng = np.random.default_rng(5)
    even = rng.integers(0, 1 << 20, 40_000)
    few = (1 << 20) + rng.integers(0, 200, 40_000) * 4000
    check(rng.permutation(np.concatenate([even, few])))
