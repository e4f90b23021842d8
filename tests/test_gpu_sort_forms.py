"""GPU parity of the radix sort where its passes change form: the tile counts at
which the passes add up all tiles themselves or take them in groups of one, two,
four and eight, device counts far below and at the capacity, digits of one to
eight bits with few distinct values, and the filtered sort over one and several
predicate columns.  Exact, against torch's stable sort."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TILE = 4096


@pytest.fixture(scope="module")
def tqp():
    import paper_2209_04579_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def ints(n, lo, hi, dtype, seed):
    return torch.randint(lo, hi, (n,), generator=gen(seed), device="cuda", dtype=torch.int64).to(dtype)


@pytest.mark.parametrize("tiles", [1, 2, 31, 32, 33, 64, 65, 2047, 2048, 4095, 4096, 8191, 8192])
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_tile_groups(tqp, tiles, extra):
    n = tiles * TILE + extra
    key = ints(n, 0, 1000, torch.int32, tiles)
    k, rows = tqp.sort(key, key_bits=10)
    want, idx = torch.sort(key, stable=True)
    assert torch.equal(k, want) and torch.equal(rows.long(), idx)


@pytest.mark.parametrize("cap", [200_000, 9_000_000, 17_000_000, 40_000_000])
@pytest.mark.parametrize("share", [0.0, 1e-6, 0.001, 0.3, 1.0])
def test_device_count_below_the_capacity(tqp, cap, share):
    n = int(cap * share)
    key = ints(cap, -500, 500, torch.int32, cap)
    pay = ints(cap, -100, 100, torch.int8, 5)
    ok, op = torch.full_like(key, 77), torch.full_like(pay, 77)
    rows = torch.full((cap,), 77, dtype=torch.int32, device="cuda")
    d_n = torch.tensor([n], dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.sort_workspace_bytes(cap, torch.int32, 1))
    for _ in range(2):
        tqp.sort_into(key, None, cap, ok, rows, ws, d_n=d_n, key_bits=10, key_min=-500, pay_in=[pay],
                      pay_out=[op])
    want, idx = torch.sort(key[:n], stable=True)
    assert torch.equal(ok[:n], want) and torch.equal(rows[:n].long(), idx) and torch.equal(op[:n], pay[:n][idx])
    assert (ok[n:] == 77).all() and (rows[n:] == 77).all() and (op[n:] == 77).all()


@pytest.mark.parametrize("bits", [1, 2, 3, 7, 8, 9, 15, 16, 17, 24, 25, 31, 32, 33, 48, 63, 64])
@pytest.mark.parametrize("few", [False, True])
def test_key_bits(tqp, bits, few):
    n = 70_003
    dt = torch.int32 if bits <= 32 else torch.int64
    key = ints(n, -(1 << 63), (1 << 63) - 1, torch.int64, bits)
    if bits < 64:
        key = (key >> 1) & ((1 << min(bits, 63)) - 1)
    if few:                              # two values, one of them almost always
        key = torch.where(key % 97 == 0, key[0], key[1])
    lo = -(1 << (bits - 1))
    key = (key + (lo if bits < 64 else 0)).to(dt)
    pay = [ints(n, -100, 100, torch.int8, 1), ints(n, 0, 1 << 40, torch.int64, 2),
           ints(n, -9, 9, torch.int32, 3), ints(n, -(1 << 50), 1 << 50, torch.int64, 4)]
    want, idx = torch.sort(key, stable=True)
    for npay in (0, 1, 4):
        for want_rows in (False, True):
            got = tqp.sort(key, key_bits=bits, key_min=lo, payload=pay[:npay], want_rows=want_rows)
            assert torch.equal(got[0], want)
            assert not want_rows or torch.equal(got[1].long(), idx)
            for p, g in zip(pay, got[2] if npay else []):
                assert torch.equal(g, p[idx])


@pytest.mark.parametrize("n", [1, 63, 64, 65, TILE - 1, TILE, TILE + 1, 131_072, 131_073, 1_000_003, 8_388_609])
def test_filtered_sort(tqp, n):
    key = ints(n, -(1 << 20), 1 << 20, torch.int64, n)
    cols = [ints(n, 0, 100, torch.int32, 1), ints(n, -50, 50, torch.int8, 2), ints(n, 0, 1 << 40, torch.int64, 3)]
    ok, rows = torch.empty_like(key), torch.empty(n, dtype=torch.int32, device="cuda")
    op = torch.empty_like(cols[1])
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.sort_workspace_bytes(n, torch.int64, 1))
    for preds, keep in (([(0, "<", 50)], cols[0] < 50), ([(0, "<", 0)], cols[0] < 0), ([(0, ">=", 0)], cols[0] >= 0),
                        ([(0, "!=", 3), (1, ">", -20), (2, "<=", 1 << 39), (1, "<", 30)],
                         (cols[0] != 3) & (cols[1] > -20) & (cols[2] <= 1 << 39) & (cols[1] < 30))):
        tqp.filter_sort_into(cols, preds, key, ok, rows, cnt, ws, key_bits=21, key_min=-(1 << 20),
                             pay_in=[cols[1]], pay_out=[op])
        at = torch.nonzero(keep).view(-1)
        want, idx = torch.sort(key[at], stable=True)
        k = int(cnt.item())
        assert k == len(at)
        assert torch.equal(ok[:k], want) and torch.equal(rows[:k].long(), at[idx]) and torch.equal(op[:k], cols[1][at[idx]])
