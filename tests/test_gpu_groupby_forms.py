"""GPU parity of the group-by's two paths where they change form: runs that end at,
begin at and cover whole blocks of rows, the row counts where a block grows, one
to four sums over few and many value columns, and dense domains from one key to
the largest, which set how many copies of each LDS cell there are.  Exact,
against the CPU oracle (tables of millions of rows: against torch)."""
import numpy as np
import pytest

import tqp_datagen as dg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

AGGS = [("sum", 0), ("sum_product", 0, 1), ("count",), ("sum_diff_product", 1, 2, 100)]


@pytest.fixture(scope="module")
def tqp():
    import paper_2209_04579_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(tqp, key, vals, aggs, **kw):
    got_k, got = tqp.groupby_agg(dev(key), [dev(v) for v in vals], aggs, **kw)
    want = groups_of(key, vals, aggs)
    assert np.array_equal(got_k.cpu().numpy(), want[0])
    for a, g, w in zip(aggs, got, want[1]):
        assert np.array_equal(g.cpu().numpy(), w), a


def groups_of(key, vals, aggs):
    # SUM_DIFF_PRODUCT is a plain product with the difference
    vals, out = [v.astype(np.int64) for v in vals], []
    for a in aggs:
        if a[0] == "sum_diff_product":
            vals.append(np.int64(a[3]) - vals[a[2]])
            out.append(("sum_product", a[1], len(vals) - 1))
        else:
            out.append(a)
    uniq, inv = np.unique(key, return_inverse=True)
    res = []
    for a in out:
        t = (np.ones(len(key), np.int64) if a[0] == "count" else
             vals[a[1]] if a[0] == "sum" else vals[a[1]] * vals[a[2]])
        s = np.zeros(len(uniq), np.int64)
        np.add.at(s, inv, t)
        res.append(s)
    return uniq, res


def values(n, seed):
    return [dg.uniform_int(seed, 1, n, -(1 << 31), 1 << 31, np.int64) * 1_000_003,
            dg.uniform_int(seed, 2, n, -100, 100, np.int8),
            dg.uniform_int(seed, 3, n, -10 ** 6, 10 ** 6, np.int32)]


# run lengths around a thread's rows, a tile (2048 rows) and several of them
@pytest.mark.parametrize("length", [1, 2, 3, 4, 5, 63, 64, 65, 255, 256, 2_047, 2_048, 2_049, 5_000, 40_000])
@pytest.mark.parametrize("dt", [np.int32, np.int64])
def test_runs_across_blocks(tqp, length, dt):
    n = 21_111
    for shift in (0, 1, 1_024):
        key = ((np.arange(n) + shift) // length - 3).astype(dt)
        check(tqp, key, values(n, 1), AGGS, flags=tqp.GB_SORTED)


@pytest.mark.parametrize("n", [0, 1, 4, 5, 2_047, 2_048, 2_049, 4_096, 4_097])
def test_ragged_ends(tqp, n):
    key = np.sort(dg.uniform_int(n, 1, n, 0, 40, np.int64) ** 2)
    check(tqp, key, values(n, n), AGGS, flags=tqp.GB_SORTED)
    check(tqp, key[::-1].copy(), values(n, n), AGGS)


@pytest.mark.parametrize("aggs", [[("count",)], [("sum", 1)], [("sum", 0), ("sum", 0)],
                                  [("sum", 0), ("sum", 1), ("sum", 2)],
                                  [("sum_product", 0, 1), ("sum_product", 1, 2), ("sum_product", 2, 0),
                                   ("sum_diff_product", 0, 1, -7)],
                                  [("count",), ("sum", 2), ("count",), ("sum_product", 2, 2)]])
@pytest.mark.parametrize("span", [1, 7, 40, 1_000])
def test_aggregates_and_domains(tqp, aggs, span):
    n = 30_001
    key = dg.uniform_int(span, 4, n, 0, span, np.int32) - 5
    vals = values(n, span)
    check(tqp, key, vals, aggs, flags=tqp.GB_DENSE, key_lo=-5, key_span=span)
    check(tqp, np.sort(key), vals, aggs, flags=tqp.GB_SORTED)
    check(tqp, key, vals, aggs)


@pytest.mark.parametrize("span", [2_047, 4_095, 4_096])
def test_largest_dense_domains(tqp, span):
    key = dg.uniform_int(9, 4, 50_003, 0, span, np.int64)
    check(tqp, key, values(50_003, 9), [("sum", 0)] if span < 4_096 else [("count",)],
          flags=tqp.GB_DENSE, key_span=span)


def test_output_smaller_than_the_groups(tqp):
    n, cap = 30_000, 100
    key, val = np.arange(n, dtype=np.int32) // 7, values(n, 2)[0]
    ok = torch.full((cap + 4,), -9, dtype=torch.int32, device="cuda")
    out = [torch.full((cap + 4,), -9, dtype=torch.int64, device="cuda") for _ in range(2)]
    ng = torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.groupby_workspace_bytes(n, torch.int32, 2, tqp.GB_SORTED))
    tqp.groupby_agg_into(dev(key), [dev(val)], [("sum", 0), ("count",)], ok[:cap], out, ng, ws,
                         flags=tqp.GB_SORTED)
    uniq, (s, c) = groups_of(key, [val], [("sum", 0), ("count",)])
    assert int(ng.item()) == len(uniq)
    for got, want in ((ok, uniq), (out[0], s), (out[1], c)):
        assert np.array_equal(got.cpu().numpy()[:cap], want[:cap])
        assert (got.cpu().numpy()[cap:] == -9).all()


@pytest.mark.parametrize("terms", [[(0, 0, 5), (None, 0, -3)], [(0, 3, 1), (1, 0, 3), (2, 4, 9)],
                                   [(1, 0, 1), (0, 7, 2), (2, 8, 40), (None, 0, 11)]])
def test_packed_keys_of_one_to_four_terms(tqp, terms):
    n = 9_011
    cols = [dg.uniform_int(3, 1, n, 0, 20, np.int8), dg.uniform_int(3, 2, n, 0, 3, np.int64),
            dg.uniform_int(3, 3, n, -50, 50, np.int32)]
    rows = dg.uniform_int(3, 4, n, 0, n, np.int32)
    key = np.zeros(n, np.int64)
    for c, mod, mul in terms:
        v = np.int64(1) if c is None else cols[c].astype(np.int64)[rows if c == 1 else slice(None)]
        key += mul * (v % mod if mod and c is not None else v)
    lo, span = int(key.min()), int(key.max() - key.min() + 1)
    vals, aggs = values(n, 6), [("sum_product", 0, 1), ("count",)]
    vrows = dg.uniform_int(3, 5, n, 0, n, np.int32)
    ok = torch.empty(span, dtype=torch.int64, device="cuda")
    out = [torch.empty(span, dtype=torch.int64, device="cuda") for _ in aggs]
    ng = torch.empty(1, dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.groupby_terms_workspace_bytes(len(aggs), span))
    tqp.groupby_agg_terms_into([(None if c is None else dev(cols[c]), dev(rows) if c == 1 else None, mod, mul)
                                for c, mod, mul in terms], n, [dev(v) for v in vals], aggs, ok, out, ng, ws,
                               lo, span, val_rows=dev(vrows))
    uniq, want = groups_of(key, [v[vrows] for v in vals], aggs)
    g = int(ng.item())
    assert np.array_equal(ok[:g].cpu().numpy(), uniq)
    for x, w in zip(out, want):
        assert np.array_equal(x[:g].cpu().numpy(), w)


# rows where a block grows from 1 to 2, 4 and 8 tiles; one key covers them all,
# then each key a few rows
@pytest.mark.parametrize("n", [(1 << 24) + d for d in (-1, 0, 2_049)] + [(1 << 25) + 3, (1 << 26) + 77])
def test_block_length_changes(tqp, n):
    val = torch.arange(n, dtype=torch.int32, device="cuda")
    for length in (n, 1_000_003, 37):
        key = torch.div(val, length, rounding_mode="floor")
        k, (s, c) = tqp.groupby_agg(key, [val], [("sum", 0), ("count",)], flags=tqp.GB_SORTED,
                                    cap=n // length + 2)
        m = -(-n // length)
        first = torch.arange(m, device="cuda") * length
        size = (first + length).clamp(max=n) - first
        assert torch.equal(k.long(), torch.arange(m, device="cuda"))
        assert torch.equal(c, size) and torch.equal(s, first * size + size * (size - 1) // 2)
