"""Ranges of a join do not depend on which side the match starts from: left longer,
right longer and equal sides, with repeated keys on both, against numpy; the pairs
expanded beside the ranges too."""
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


@pytest.mark.parametrize("dt", [np.int32, np.int64])
@pytest.mark.parametrize("nl,nr", [(1, 1), (7, 3), (3, 7), (1025, 1024), (1024, 1025), (60_001, 900), (900, 60_001),
                                   (0, 5), (5, 0)])
def test_ranges_from_either_side(tqp, dt, nl, nr):
    rng = np.random.default_rng(nl * 7 + nr)
    span = max(2, min(nl, nr))
    lk, rk = (np.sort(rng.integers(-span, span, n)).astype(dt) for n in (nl, nr))
    ul, ls, lc = np.unique(lk, return_index=True, return_counts=True)
    ur, rs, rc = np.unique(rk, return_index=True, return_counts=True)
    key, il, ir = np.intersect1d(ul, ur, return_indices=True)
    want = [key, ls[il], lc[il], rs[ir], rc[ir]]
    m, total = len(key), int((lc[il] * rc[ir]).sum())
    dl, dr = torch.from_numpy(lk).cuda(), torch.from_numpy(rk).cuda()
    flags = tqp.JOIN_SORTED | tqp.JOIN_RANGES
    for cap in (0, total + 3, total // 2):
        ranges = [torch.full((max(m, 1),), -9, dtype=torch.int64, device="cuda") for _ in range(5)]
        ol, orr = (torch.full((max(cap, 1),), -5, dtype=torch.int32, device="cuda") for _ in range(2))
        cnt, nrg = (torch.zeros(1, dtype=torch.int64, device="cuda") for _ in range(2))
        ws = tqp.workspace(tqp.join_workspace_bytes(nl, nr, dl.dtype, flags, cap))
        tqp.join_into(dl, dr, flags, ol if cap else None, orr if cap else None, None, cap, cnt, ws,
                      ranges=ranges, range_cap=max(m, 1), d_nranges=nrg)
        assert int(cnt.item()) == total and int(nrg.item()) == m
        for got, w in zip(ranges, want):
            assert np.array_equal(got[:m].cpu().numpy(), w)
        if cap:
            i = np.concatenate([np.repeat(np.arange(a, a + b), d) for _, a, b, c, d in zip(*want)] or [[]])
            j = np.concatenate([np.tile(np.arange(c, c + d), b) for _, a, b, c, d in zip(*want)] or [[]])
            k = min(cap, total)
            assert np.array_equal(ol[:k].cpu().numpy(), i[:k]) and np.array_equal(orr[:k].cpu().numpy(), j[:k])
