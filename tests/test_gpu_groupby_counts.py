"""GPU parity of the dense group-by that only counts, where a workgroup's share of the rows
follows the number of keys (sixteen rows per key, from 129 keys on): around whole shares,
and with the row count on the device.  Exact against torch."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kdt", ["int32", "int64"])
@pytest.mark.parametrize("span", [1, 127, 128, 129, 1500, 3072])
@pytest.mark.parametrize("shares,rest", [(0, 0), (0, 1), (1, -1), (1, 0), (1, 1), (37, 5), (513, 1)])
def test_counts(span, shares, rest, kdt):
    import paper_2209_04579_amd as tqp
    n = shares * max(2048, 16 * span) + rest
    g = torch.Generator(device="cuda").manual_seed(n % 1000 + span)
    key = torch.randint(0, span, (n + 7,), device="cuda", generator=g).to(getattr(torch, kdt))
    key = key[: n if shares != 37 else n + 7]
    ws = tqp.workspace(tqp.groupby_workspace_bytes(key.numel(), key.dtype, 1, 2, span))
    ok = torch.zeros(span, dtype=key.dtype, device="cuda")
    cnt = torch.zeros(span, dtype=torch.int64, device="cuda")
    ng = torch.empty(1, dtype=torch.int64, device="cuda")
    d_n = torch.tensor([n], dtype=torch.int64, device="cuda") if key.numel() > n else None
    tqp.groupby_agg_into(key, [], [("count",)], ok, [cnt], ng, ws, flags=2, key_lo=0, key_span=span, d_n=d_n)
    want = torch.bincount(key[:n].long(), minlength=span)
    keys = torch.nonzero(want).flatten()
    m = int(ng.item())
    assert m == keys.numel()
    assert torch.equal(ok[:m].long(), keys) and torch.equal(cnt[:m], want[keys])
