"""GPU parity of the semi-join scan where its forms change: key ranges that begin
below, end above, lie outside or cover the whole of int32 (positions are computed
modulo 2^32 there), several tiles per workgroup, and tiles that keep few, many, all
and none of their rows side by side.  Exact against a numpy look-up."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MIN, MAX = -2**31, 2**31 - 1


@pytest.fixture(scope="module")
def tqp():
    import paper_2209_04579_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def keyset(tqp, keys, lo, nb):
    bits = torch.empty(max(tqp.keyset_words(nb), 1), dtype=torch.int32, device="cuda")
    tqp.keyset_build_into(torch.from_numpy(np.asarray(keys)).cuda(), lo, nb, bits)
    return bits, lo, nb


def scan(tqp, keys, sets, want, pay=None):
    n = len(keys[0])
    dk = [torch.from_numpy(k).cuda() for k in keys]
    rows = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    kout = [torch.zeros_like(k) for k in dk]
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    pin = [torch.from_numpy(pay).cuda()] if pay is not None else []
    pout = [torch.zeros_like(p) for p in pin]
    ws = tqp.workspace(tqp.semijoin_workspace_bytes(n, dk[0].dtype))
    for _ in range(2):
        tqp.semijoin_into(dk, sets, rows, cnt, ws, keys_out=kout, payload_in=pin, payload_out=pout)
    k = int(cnt.item())
    assert k == len(want) and np.array_equal(rows[:k].cpu().numpy(), want)
    for src, got in zip(keys, kout):
        assert np.array_equal(got[:k].cpu().numpy(), src[want])
    for got in pout:
        assert np.array_equal(got[:k].cpu().numpy(), pay[want])


@pytest.mark.parametrize("lo,nb", [(MIN - 45, 100), (MIN - 64, 96), (MIN - 45, 1 << 21), (MIN, 64), (MAX - 10, 1000),
                                   (MAX - 40, 41), (MAX + 1, 500), (MIN - 500, 500), (-2**40, 77),
                                   (MIN, 1 << 32), (MIN - 7, (1 << 32) + 50), (5, 0)])
def test_ranges_at_the_ends_of_int32(tqp, lo, nb):
    rng = np.random.default_rng(abs(lo) % 1000 + nb % 1000)
    near = np.concatenate([MIN + np.arange(90), MAX - np.arange(90), np.arange(-5, 5),
                           rng.integers(MIN, MAX, 3000)]).astype(np.int64)
    keys = rng.permutation(np.concatenate([near, near[::2]])).astype(np.int32)
    pool = np.unique(np.concatenate([near[::2], lo + np.arange(min(nb, 200))[::2]])).astype(np.int64)
    member = pool[(pool >= lo) & (pool - lo < nb)]
    want = np.flatnonzero(np.isin(keys.astype(np.int64), member)).astype(np.int32)
    scan(tqp, [keys], [keyset(tqp, pool, lo, nb)], want)
    # beside a set on chip
    other = (np.abs(keys.astype(np.int64)) % 50).astype(np.int32)
    keep = np.flatnonzero(np.isin(keys.astype(np.int64), member) & (other < 25)).astype(np.int32)
    scan(tqp, [other, keys], [keyset(tqp, np.arange(25), 0, 50), keyset(tqp, pool, lo, nb)], keep)


@pytest.mark.parametrize("kdt", [np.int32, np.int64])
@pytest.mark.parametrize("ns", [1, 2, 3, 4])
@pytest.mark.parametrize("mem", [False, True])
def test_tiles_of_every_density(tqp, kdt, ns, mem):
    n, size = 8_500_001, 1000
    rng = np.random.default_rng(ns)
    member = np.zeros(size, bool)
    member[:500] = True
    keys = [np.full(n, 700, kdt) for _ in range(ns)]
    for beg, end, share in ((0, 3_000_000, 0.003), (3_000_000, 3_100_000, 1.0), (3_100_000, 3_700_000, 0.3),
                            (5_000_000, 5_000_003, 1.0), (7_000_000, n, 0.02)):
        hit = beg + np.flatnonzero(rng.random(end - beg) < share)
        for k in keys:
            k[hit] = rng.integers(0, 501, len(hit))       # 500 is not a member
    if n:
        for k in keys:
            k[-1] = 3
    ok = member[keys[0].astype(np.int64)]
    for k in keys[1:]:
        ok &= member[k.astype(np.int64)]
    want = np.flatnonzero(ok).astype(np.int32)
    pay = rng.integers(-100, 100, n).astype(np.int8)
    sets = [keyset(tqp, np.arange(500), 0, size) for _ in range(ns)]
    if mem:                                    # a range too wide for the chip
        sets[-1] = keyset(tqp, np.arange(500), -40_000_000, 80_000_000)
    scan(tqp, keys, sets, want, pay)


def test_parts_of_the_static_scratch(tqp):
    n = 2 * (1 << 25) + 70_003                 # three parts
    g = torch.Generator(device="cuda").manual_seed(5)
    keys = [torch.randint(0, s, (n,), device="cuda", dtype=torch.int32, generator=g) for s in (100, 7)]
    keys[0][:40_000_000:3] = 1000              # few in the first part
    ok = (keys[0] < 30) & (keys[1] < 2)
    want = torch.nonzero(ok).flatten().int()
    sets = [keyset(tqp, np.arange(30), 0, 100), keyset(tqp, np.arange(2), 0, 7)]
    pay = torch.randint(-100, 100, (n,), device="cuda", dtype=torch.int8, generator=g)
    rows = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    kout, pout = [torch.zeros_like(k) for k in keys], torch.zeros_like(pay)
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    for _ in range(2):
        tqp.semijoin_noalloc_into(keys, sets, rows, cnt, keys_out=kout, payload_in=[pay], payload_out=[pout])
    k = int(cnt.item())
    assert k == want.numel() and torch.equal(rows[:k], want) and int((rows[k:] + 7).abs().sum()) == 0
    for src, got in zip(keys + [pay], kout + [pout]):
        assert torch.equal(got[:k], src[want.long()])
