"""GPU parity of the join's pairs where the kernels change form: tiles of left rows
with and without matches, right windows inside and beyond what is staged, right
rows unique, repeated and so often repeated that a tile's pairs are spread over
the chip, output capacities below the total, device counts, and left sides long
enough for several tiles per block.  Exact, in order, against numpy."""
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


def pairs_of(lk, rk):
    """(i, j) of every pair over two sorted sides, by left row then right row (device tensors)."""
    lo, hi = torch.searchsorted(rk, lk), torch.searchsorted(rk, lk, right=True)
    m = hi - lo
    i = torch.repeat_interleave(torch.arange(len(lk), device="cuda"), m)
    first = torch.cumsum(m, 0) - m
    return i, lo[i] + torch.arange(len(i), device="cuda") - first[i]


def check(tqp, lk, rk, lrows=None, rrows=None, cap=None):
    i, j = pairs_of(lk, rk)
    total = len(i)
    cap = total + 7 if cap is None else cap
    ol, orr = (torch.full((max(cap, 1),), -5, dtype=torch.int32, device="cuda") for _ in range(2))
    ok = torch.full((max(cap, 1),), -5, dtype=lk.dtype, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.join_workspace_bytes(len(lk), len(rk), lk.dtype, tqp.JOIN_SORTED, cap))
    for _ in range(2):
        tqp.join_into(lk, rk, tqp.JOIN_SORTED, ol, orr, ok, cap, cnt, ws, lrows=lrows, rrows=rrows)
    assert int(cnt.item()) == total
    m = min(total, cap)
    i, j = i[:m], j[:m]
    assert torch.equal(ok[:m], lk[i])
    assert torch.equal(ol[:m].long(), i if lrows is None else lrows[i].long())
    assert torch.equal(orr[:m].long(), j if rrows is None else rrows[j].long())
    for o in (ol, orr, ok):
        assert (o[m:] == -5).all()


def sorted_keys(n, lo, hi, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.sort(torch.randint(lo, hi, (n,), generator=g, device="cuda", dtype=torch.int64))[0].to(dtype)


@pytest.mark.parametrize("dt", [torch.int32, torch.int64])
@pytest.mark.parametrize("nl", [1, 7, 2047, 2048, 2049, 40_001])
@pytest.mark.parametrize("nr", [1, 63, 64, 65, 2048, 4097, 50_000])
def test_sizes_and_windows(tqp, dt, nl, nr):
    for span in (3, 300, 5_000, 1_000_000):
        lk, rk = sorted_keys(nl, -span, span, dt, nl + span), sorted_keys(nr, -span, span, dt, nr + span)
        if nl * nr // span < 40_000_000:
            check(tqp, lk, rk)


@pytest.mark.parametrize("dt", [torch.int32, torch.int64])
def test_unique_right_side_with_gaps(tqp, dt):
    rk = (torch.arange(100_000, device="cuda") * 3).to(dt)
    rows = torch.randperm(100_000, device="cuda").to(torch.int32)
    for step in (1, 2, 3, 100, 290):                      # right rows skipped per left row
        lk = (torch.arange(1, 300_000 // step, device="cuda") * step).to(dt)
        check(tqp, lk, rk, lrows=rows[:1].expand(len(lk)).contiguous(), rrows=rows)
    check(tqp, rk[:0], rk), check(tqp, rk, rk[:0]), check(tqp, rk + 1, rk), check(tqp, rk[50_000:], rk[:50_000])


@pytest.mark.parametrize("hot_l,hot_r", [(1, 20_000), (20_000, 1), (2_048, 9), (2_048, 8), (3_000, 3_000), (5, 400_000)])
def test_hot_keys(tqp, hot_l, hot_r):
    # keys below, a hot key, keys above; then several hot keys in one tile
    for hots in ([500], [100, 101, 800]):
        base = torch.arange(0, 1000, 7, device="cuda")
        l, r = [base], [base]
        for h in hots:
            l.append(torch.full((hot_l,), h, device="cuda"))
            r.append(torch.full((hot_r,), h, device="cuda"))
        lk, rk = (torch.sort(torch.cat(x))[0].to(torch.int32) for x in (l, r))
        check(tqp, lk, rk)


@pytest.mark.parametrize("cap", [0, 1, 5_000, 100_000, 4_999_999])
def test_capacity_below_the_total(tqp, cap):
    lk = sorted_keys(20_000, 0, 40, torch.int32, 1)
    rk = sorted_keys(10_000, 0, 40, torch.int32, 2)
    check(tqp, lk, rk, cap=cap)


def test_device_counts(tqp):
    lk, rk = sorted_keys(50_000, 0, 9_000, torch.int64, 3), sorted_keys(30_000, 0, 9_000, torch.int64, 4)
    ws = tqp.workspace(tqp.join_workspace_bytes(50_000, 30_000, torch.int64, tqp.JOIN_SORTED, 400_000))
    ol, orr = (torch.empty(400_000, dtype=torch.int32, device="cuda") for _ in range(2))
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    for nl, nr in ((0, 30_000), (50_000, 0), (1, 1), (2_049, 30_000), (50_000, 777), (60_000, 30_000)):
        d = torch.tensor([nl, nr], dtype=torch.int64, device="cuda")
        tqp.join_into(lk, rk, tqp.JOIN_SORTED, ol, orr, None, 400_000, cnt, ws, d_nl=d[:1], d_nr=d[1:])
        i, j = pairs_of(lk[:nl], rk[:nr])
        assert int(cnt.item()) == len(i)
        assert torch.equal(ol[:len(i)].long(), i) and torch.equal(orr[:len(i)].long(), j)


@pytest.mark.parametrize("nl", [(1 << 22) + 3, (1 << 23) + 1, (1 << 24) + 2_049, (1 << 25) + 7])
def test_several_tiles_per_block(tqp, nl):
    for nr, span in ((100_000, 400_000), (3_000_000, 40_000_000)):
        check(tqp, sorted_keys(nl, 0, span, torch.int32, 5), sorted_keys(nr, 0, span, torch.int32, 6))
