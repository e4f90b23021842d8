"""Joins whose output capacity is within what a tile's own workgroup writes: tiles of
very many pairs cut off at the capacity, counts whole."""
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


@pytest.mark.parametrize("cap", [1, 5000, 16383, 16384, 16385])
@pytest.mark.parametrize("nl,nr,vals", [(300, 200, 1), (4100, 5000, 2), (5000, 4100, 700), (9000, 1 << 20, 3)])
def test_capacity_below_a_tiles_pairs(tqp, cap, nl, nr, vals):
    rng = np.random.default_rng(nl)
    lk, rk = np.sort(rng.integers(0, vals, nl)).astype(np.int32), np.sort(rng.integers(0, vals, nr)).astype(np.int32)
    lo, hi = np.searchsorted(rk, lk), np.searchsorted(rk, lk, side="right")
    off = np.concatenate([[0], np.cumsum(hi - lo)])
    total, k = int(off[-1]), min(cap, int(off[-1]))
    row = np.searchsorted(off, np.arange(k), side="right") - 1
    ol, orr = (torch.full((cap + 9,), -5, dtype=torch.int32, device="cuda") for _ in range(2))
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.join_workspace_bytes(nl, nr, torch.int32, tqp.JOIN_SORTED, cap))
    tqp.join_into(torch.from_numpy(lk).cuda(), torch.from_numpy(rk).cuda(), tqp.JOIN_SORTED, ol, orr, None, cap, cnt,
                  ws)
    assert int(cnt.item()) == total
    assert np.array_equal(ol[:k].cpu().numpy(), row)
    assert np.array_equal(orr[:k].cpu().numpy(), lo[row] + np.arange(k) - off[row])
    assert (ol[k:] == -5).all() and (orr[k:] == -5).all()
