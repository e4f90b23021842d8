"""Unsorted group-by of a million rows and more, where up to two value columns move
along with the keys through the sort: every mix of value types, key widths on both
sides of the rule, rows given by id and fewer rows than capacity; columns shorter
than the capacity are refused as ever.  Exact against torch."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROWS = 1 << 20


@pytest.fixture(scope="module")
def tqp():
    import paper_2209_04579_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


I8, I32, I64 = torch.int8, torch.int32, torch.int64


FORMS = [("plain", n, k) for n in (ROWS - 1, ROWS, ROWS + 4097) for k in ((I32, 1 << 16), (I64, 1 << 30), (I64, 1 << 62))]
FORMS += [(form, ROWS + 4097, k) for form in ("d_n", "rows") for k in ((I32, 1 << 16), (I64, 1 << 62))]


@pytest.mark.parametrize("form,n,keys", FORMS)
@pytest.mark.parametrize("vdt", [(I64,), (I8,), (I64, I8), (I64, I64), (I32, I32), (I64, I32, I8)])
def test_carried_values(tqp, form, n, keys, vdt):
    kdt, span = keys
    g = torch.Generator(device="cuda").manual_seed(n % 97 + span % 89 + len(vdt))
    pool = torch.randint(-span // 2, span // 2, (50_000,), device="cuda", dtype=I64, generator=g)
    key = pool[torch.randint(0, 50_000, (n,), device="cuda", generator=g)].to(kdt)
    cnt = n - 300_001 if form == "d_n" else n
    vals = [torch.randint(-120, 121, (n,), device="cuda", generator=g).to(d) for d in vdt]
    rows = torch.randperm(n, device="cuda", generator=g).to(I32) if form == "rows" else None
    d_n = torch.tensor([cnt], dtype=I64, device="cuda") if cnt < n else None
    aggs = [("sum", len(vdt) - 1), ("sum_product", 0, len(vdt) - 1), ("count",)]
    ok = torch.zeros(n, dtype=kdt, device="cuda")
    out = [torch.zeros(n, dtype=I64, device="cuda") for _ in aggs]
    ng = torch.zeros(1, dtype=I64, device="cuda")
    ws = tqp.workspace(tqp.groupby_workspace_bytes(n, kdt, len(aggs), 0, 0))
    tqp.groupby_agg_into(key, vals, aggs, ok, out, ng, ws, val_rows=rows, d_n=d_n)
    if form == "d_n":
        with pytest.raises(tqp.TqpError):
            tqp.groupby_agg_into(key, [c[:cnt] for c in vals], aggs, ok, out, ng, ws, d_n=d_n)
    at = rows[:cnt].long() if rows is not None else torch.arange(cnt, device="cuda")
    uniq, inv = torch.unique(key[:cnt], return_inverse=True)
    v = [c[at].to(I64) for c in vals]
    want = [torch.zeros(len(uniq), dtype=I64, device="cuda").index_add_(0, inv, x)
            for x in (v[-1], v[0] * v[-1], torch.ones(cnt, dtype=I64, device="cuda"))]
    m = int(ng.item())
    assert m == len(uniq) and torch.equal(ok[:m], uniq)
    for got, w in zip(out, want):
        assert torch.equal(got[:m], w)
