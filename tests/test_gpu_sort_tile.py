"""Sorts of at most one tile run in one launch: sizes around waves and the tile, digit
widths from one bit to eight passes, signed extremes, equal keys, row ids given or
not, payload of every type, and counts below the capacity.  Exact against a
stable sort."""
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


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 1025, 4095, 4096, 4097])
@pytest.mark.parametrize("dt,bits", [(np.int32, 1), (np.int32, 11), (np.int32, 32), (np.int64, 8), (np.int64, 41),
                                     (np.int64, 64)])
@pytest.mark.parametrize("short", [False, True])
def test_one_tile(tqp, n, dt, bits, short):
    rng = np.random.default_rng(n * 100 + bits)
    lo = -(1 << (bits - 1))
    key = rng.integers(lo, -lo, n, dtype=np.int64, endpoint=False) if bits > 1 else rng.integers(-1, 1, n)
    key[: n // 3] = key[n // 2]                       # equal keys
    key[0], key[-1] = -lo - 1 if bits > 1 else 0, lo
    key = key.astype(dt)
    pay = [rng.integers(-100, 100, n).astype(t) for t in (np.int8, np.int64, np.int32)]
    rows = rng.permutation(n).astype(np.int32)
    cnt = max(n - 7, 0) if short else n
    d_n = torch.tensor([cnt], dtype=torch.int64, device="cuda") if short else None
    dev = [torch.from_numpy(a).cuda() for a in (key, rows, *pay)]
    order = np.argsort(key[:cnt], kind="stable")
    for given in (True, False):
        ok = torch.full((n,), 5, dtype=dev[0].dtype, device="cuda")
        orow = torch.full((n,), -9, dtype=torch.int32, device="cuda")
        po = [torch.full_like(p, 77) for p in dev[2:]]
        ws = tqp.workspace(tqp.sort_workspace_bytes(n, dev[0].dtype, 13))
        tqp.sort_into(dev[0], dev[1] if given else None, n, ok, orow, ws, d_n=d_n, key_bits=bits, key_min=lo,
                      pay_in=dev[2:], pay_out=po)
        assert np.array_equal(ok.cpu().numpy()[:cnt], key[:cnt][order])
        assert (ok.cpu().numpy()[cnt:] == 5).all() and (orow.cpu().numpy()[cnt:] == -9).all()
        assert np.array_equal(orow.cpu().numpy()[:cnt], rows[order] if given else order)
        for p, got in zip(pay, po):
            assert np.array_equal(got.cpu().numpy()[:cnt], p[order]) and (got.cpu().numpy()[cnt:] == 77).all()
