"""Ranges of a join where the side with fewer rows has more runs and the other way round: the
match starts from the side with fewer runs.  Exact against torch."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.int32, torch.int64])
@pytest.mark.parametrize("nl,kl,nr,kr", [(50_000, 3, 20_000, 1 << 28), (20_000, 1 << 28, 50_000, 3),
                                         (50_000, 1 << 28, 20_000, 3), (30_000, 1024, 30_000, 1025),
                                         (5000, 1, 4000, 4000), (4000, 4000, 5000, 1), (300_000, 2000, 100_000, 90_000),
                                         (0, 1, 10, 5), (10, 5, 0, 1)])
@pytest.mark.parametrize("d_n", [False, True])
def test_match_from_the_side_of_fewer_runs(dt, nl, kl, nr, kr, d_n):
    import paper_2209_04579_amd as tqp
    g = torch.Generator(device="cuda").manual_seed(nl + kr)
    l, r = (torch.sort(torch.randint(0, k, (n,), device="cuda", generator=g))[0].to(dt) for n, k in ((nl, kl), (nr, kr)))
    ml, mr = (2 * nl // 3, nr // 2) if d_n else (nl, nr)
    ul, lc = torch.unique_consecutive(l[:ml], return_counts=True)
    ur, rc = torch.unique_consecutive(r[:mr], return_counts=True)
    ls, rs = torch.cumsum(lc, 0) - lc, torch.cumsum(rc, 0) - rc
    at = torch.searchsorted(ur, ul).clamp(max=max(ur.numel() - 1, 0))
    hit = (ur[at] == ul).nonzero().flatten() if ur.numel() else at[:0]
    at = at[hit]
    want = [ul[hit].long(), ls[hit], lc[hit], rs[at], rc[at]]
    m, total = hit.numel(), int((lc[hit] * rc[at]).sum())
    cap = max(min(nl, nr), 1)
    ranges = [torch.full((cap,), -9, dtype=torch.int64, device="cuda") for _ in range(5)]
    cnt, nrg = (torch.empty(1, dtype=torch.int64, device="cuda") for _ in range(2))
    dl, dr = (torch.tensor([k], dtype=torch.int64, device="cuda") for k in (ml, mr)) if d_n else (None, None)
    flags = tqp.JOIN_SORTED | tqp.JOIN_RANGES
    ws = tqp.workspace(tqp.join_workspace_bytes(nl, nr, dt, flags, 0))
    tqp.join_into(l, r, flags, None, None, None, 0, cnt, ws, d_nl=dl, d_nr=dr, ranges=ranges, range_cap=cap, d_nranges=nrg)
    assert int(cnt.item()) == total and int(nrg.item()) == m
    for got, w in zip(ranges, want):
        assert torch.equal(got[:m], w)
