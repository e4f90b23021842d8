"""Two-class models over int32 features have a kernel instance per feature
count that scores two rows per thread: every count, sizes around its tile of
512 rows, columns of different lengths reached through row ids, and values
over the whole int32 range."""
import numpy as np
import pytest

import oracle
import tqp_datagen as dg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tqp():
    import paper_2209_04579_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("F", range(1, 17))
@pytest.mark.parametrize("n", [1, 511, 513, 70_001])
def test_two_classes_over_int32(tqp, F, n):
    H = 1 + 5 * F % 64
    model = dg.mlp_model(F, F, H, 2)
    lens = [n + (k % 3) * 7 for k in range(F)]
    lim = [30, 1 << 15, 2**31 - 1]
    feats = [dg.uniform_int(F, 20 + k, lens[k], -lim[k % 3], lim[k % 3], np.int64).astype(np.int32)
             for k in range(F)]
    out = torch.full((n + 8,), -1, dtype=torch.int8, device="cuda")
    cols, m = [dev(f) for f in feats], dev(model)
    tqp.mlp_predict_into(cols, m, H, 2, out, n=n)
    got = out.cpu().numpy()
    assert np.array_equal(got[:n], oracle.mlp_predict([f[:n] for f in feats], model, H, 2))
    assert (got[n:] == -1).all()
    # by row id: a row outside a column counts as zero there
    rows = dg.uniform_int(F, 99, n, -3, n + 20, np.int64).astype(np.int32)
    padded = [np.concatenate([np.zeros(3, np.int32), f, np.zeros(40, np.int32)]) for f in feats]
    out.fill_(-1)
    d_n = torch.tensor([max(n - 1, 1)], dtype=torch.int64, device="cuda")
    tqp.mlp_predict_into(cols, m, H, 2, out, n=n, rows=dev(rows), d_n=d_n)
    got, k = out.cpu().numpy(), max(n - 1, 1)
    want = oracle.mlp_predict([p[rows + 3] for p in padded], model, H, 2)
    assert np.array_equal(got[:k], want[:k])
    assert (got[k:] == -1).all()
