"""GPU parity of the pair join where left rows meet many right rows: pair counts per tile
of 2048 left rows around the 8192 that its own workgroup writes, chunks of 2048 pairs cut
by a run, by the tile's end or by the capacity, and windows too long for LDS whose
keys repeat.  Exact against torch, in the order (key, left, right)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TILE, DIRECT, CHUNK = 2048, 8192, 2048


def pairs(l, r):
    """Left and right positions of every pair of two ascending columns."""
    lo = torch.searchsorted(r, l)
    n = torch.searchsorted(r, l, right=True) - lo
    i = torch.repeat_interleave(torch.arange(l.numel(), device="cuda"), n)
    j = torch.arange(i.numel(), device="cuda") - torch.repeat_interleave(torch.cumsum(n, 0) - n, n) + lo[i]
    return i, j


def check(l, r, cap=None, rows=True, **kw):
    import paper_2209_04579_amd as tqp
    wi, wj = pairs(l, r)
    total = wi.numel()
    cap = total + 5 if cap is None else cap
    g = torch.Generator(device="cuda").manual_seed(9)
    lrows = torch.randperm(l.numel(), device="cuda", generator=g).int() if rows else None
    rrows = torch.randperm(r.numel(), device="cuda", generator=g).int() if rows else None
    ol, orr = (torch.full((cap + 3,), -9, dtype=torch.int32, device="cuda") for _ in range(2))
    ok = torch.full((cap + 3,), -9, dtype=l.dtype, device="cuda")
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.join_workspace_bytes(l.numel(), r.numel(), l.dtype, tqp.JOIN_SORTED, cap))
    for _ in range(2):
        tqp.join_into(l, r, tqp.JOIN_SORTED, ol, orr, ok, cap, cnt, ws, lrows=lrows, rrows=rrows, **kw)
    assert int(cnt.item()) == total
    m = min(total, cap)
    wi, wj = wi[:m], wj[:m]
    assert torch.equal(ok[:m], l[wi])
    assert torch.equal(ol[:m], lrows[wi] if rows else wi.int())
    assert torch.equal(orr[:m], rrows[wj] if rows else wj.int())
    for o in (ol, orr, ok):
        assert bool((o[m:] == -9).all())


def col(v, dt):
    return torch.sort(v)[0].to(dt)


@pytest.mark.parametrize("dt", [torch.int32, torch.int64])
@pytest.mark.parametrize("per", [3, 4, 5, 37, 5000])
@pytest.mark.parametrize("nl", [1, 7, TILE - 1, TILE, TILE + 1, 9 * TILE + 13])
def test_each_left_row_meets_many(dt, per, nl):
    if nl * per > 40_000_000:
        nl = 40_000_000 // per
    check(torch.arange(nl, device="cuda").to(dt), torch.arange(nl, device="cuda").repeat_interleave(per).to(dt))


@pytest.mark.parametrize("dt", [torch.int32, torch.int64])
@pytest.mark.parametrize("total", [DIRECT - 1, DIRECT, DIRECT + 1, DIRECT + CHUNK, 8 * CHUNK, 8 * CHUNK + 1])
def test_around_the_pairs_of_one_workgroup(dt, total):
    # one left row with most of the pairs between rows with none and with one
    l = torch.arange(0, 900, device="cuda")
    r = torch.cat([torch.full((total - 400,), 500, device="cuda"), torch.arange(1, 799, 2, device="cuda"),
                   torch.tensor([899], device="cuda")])
    check(col(l, dt), col(r, dt))


@pytest.mark.parametrize("cap", [0, 1, CHUNK - 1, CHUNK, 8 * CHUNK, 8 * CHUNK + 1, 20_480, 99_999])
@pytest.mark.parametrize("rows", [False, True])
def test_capacities_inside_a_chunk(cap, rows):
    g = torch.Generator(device="cuda").manual_seed(cap)
    l = col(torch.randint(0, 40, (5000,), device="cuda", generator=g), torch.int32)
    r = col(torch.randint(0, 40, (3000,), device="cuda", generator=g), torch.int32)
    check(l, r, cap=cap, rows=rows)


@pytest.mark.parametrize("dt", [torch.int32, torch.int64])
@pytest.mark.parametrize("nl,nr,keys", [(3000, 400_000, 2000), (10_000, 300_000, 250_000), (2000, 100_000, 3),
                                        (300_000, 3000, 100), (40_000, 40_000, 900), (1_000_000, 3_000_000, 600_000)])
def test_random_runs_on_both_sides(dt, nl, nr, keys):
    g = torch.Generator(device="cuda").manual_seed(nl)
    l = col(torch.randint(0, keys, (nl,), device="cuda", generator=g), dt)
    r = col(torch.randint(0, keys, (nr,), device="cuda", generator=g), dt)
    check(l, r, rows=nl < 1_000_000)


def test_extreme_keys_and_counts_on_the_device():
    lim = 2**63
    l = torch.tensor([-lim] * 700 + [0] * 3 + [lim - 1] * 1500, device="cuda")
    r = torch.tensor([-lim] * 300 + [5] + [lim - 1] * 6000, device="cuda")
    check(l, r)
    d = torch.tensor([2000], dtype=torch.int64, device="cuda")
    import paper_2209_04579_amd as tqp
    cap = 10_000_000
    o = [torch.empty(cap, dtype=torch.int32, device="cuda") for _ in range(2)]
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.join_workspace_bytes(l.numel(), r.numel(), l.dtype, tqp.JOIN_SORTED, cap))
    tqp.join_into(l, r, tqp.JOIN_SORTED, *o, None, cap, cnt, ws, d_nl=d)
    wi, wj = pairs(l[:2000], r)
    assert int(cnt.item()) == wi.numel()
    assert torch.equal(o[0][:wi.numel()], wi.int()) and torch.equal(o[1][:wi.numel()], wj.int())


def test_replayed_from_a_graph():
    import paper_2209_04579_amd as tqp
    g = torch.Generator(device="cuda").manual_seed(3)
    cap = 2_000_000
    l, r = (torch.zeros(n, dtype=torch.int32, device="cuda") for n in (30_000, 20_000))
    o = [torch.empty(cap, dtype=torch.int32, device="cuda") for _ in range(2)]
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.join_workspace_bytes(l.numel(), r.numel(), l.dtype, tqp.JOIN_SORTED, cap))
    graph = tqp.batch_capture(lambda: tqp.join_into(l, r, tqp.JOIN_SORTED, *o, None, cap, cnt, ws))
    for keys in (1000, 20_000, 400, 1000):
        l.copy_(col(torch.randint(0, keys, (l.numel(),), device="cuda", generator=g), torch.int32))
        r.copy_(col(torch.randint(0, keys, (r.numel(),), device="cuda", generator=g), torch.int32))
        graph.run()
        wi, wj = pairs(l, r)
        m = min(cap, wi.numel())
        assert int(cnt.item()) == wi.numel()
        assert torch.equal(o[0][:m], wi[:m].int()) and torch.equal(o[1][:m], wj[:m].int())
