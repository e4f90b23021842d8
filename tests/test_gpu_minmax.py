"""Key ranges: a column's min and max at sizes around the kernel's blocks, with
the extremes at either end, and sorts and joins that derive the range of one or
two columns from partial results."""
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


def column(n, dt, at):
    lo, hi = (np.iinfo(dt).min, np.iinfo(dt).max)
    k = np.random.default_rng(n).integers(-50, 50, n, dtype=np.int64).astype(dt)
    k[0 if at == "front" else n - 1] = lo
    if n > 1:
        k[1 if at == "front" else n - 2] = hi
    return k


@pytest.mark.parametrize("dt", [np.int8, np.int32, np.int64])
@pytest.mark.parametrize("n", [1, 2, 1023, 8193, 4_194_305])
@pytest.mark.parametrize("at", ["front", "back"])
def test_minmax(tqp, dt, n, at):
    k = column(n, dt, at)
    t = torch.from_numpy(k).cuda()
    got = torch.empty(2, dtype=torch.int64, device="cuda")
    for cnt in (n, n - 1, 0):
        d_n = torch.tensor([cnt], dtype=torch.int64, device="cuda")
        tqp.minmax_into(t, got, d_n=d_n)
        want = [int(k[:cnt].min()), int(k[:cnt].max())] if cnt else [2**63 - 1, -2**63]
        assert got.tolist() == want


@pytest.mark.parametrize("dt", [np.int32, np.int64])
@pytest.mark.parametrize("nl,nr", [(1, 1), (0, 5), (5000, 1), (3, 70_001), (1_048_577, 4097)])
def test_join_derives_both_ranges(tqp, dt, nl, nr):
    rng = np.random.default_rng(nl + nr)
    lk = rng.integers(-40, 400_000, nl).astype(dt)
    rk = rng.permutation(np.arange(-20, nr - 20)).astype(dt)
    if nr > 1:
        rk[-1] = np.iinfo(dt).max
    pl, pr = tqp.join(torch.from_numpy(lk).cuda(), torch.from_numpy(rk).cuda())
    pl, pr = pl.cpu().numpy(), pr.cpu().numpy()
    pos = {int(v): i for i, v in enumerate(rk)}
    want = sorted((i, pos[int(v)]) for i, v in enumerate(lk) if int(v) in pos)
    assert sorted(zip(pl.tolist(), pr.tolist())) == want
