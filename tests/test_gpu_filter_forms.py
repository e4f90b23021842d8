"""GPU parity of the predicate forms behind the filter and the fused filter +
aggregate: every operator with literals at and outside the limits of each column
type, contradictions, more columns than are loaded together, payload counts on
both sides of a group of four, unaligned columns, and the table sizes where a
block of rows changes its length.  Exact, against the CPU oracle."""
import numpy as np
import pytest

import oracle
import tqp_datagen as dg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DTS = [np.int8, np.int32, np.int64]
OPS = ["<", "<=", ">", ">=", "==", "!="]


@pytest.fixture(scope="module")
def tqp():
    import paper_2209_04579_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(tqp, cols, preds, payload=(), dcols=None):
    dcols = dcols or [dev(c) for c in cols]
    rows, pay = tqp.filter(dcols, preds, payload=[dev(p) for p in payload])
    want = oracle.filter_rows(cols, preds)
    assert np.array_equal(rows.cpu().numpy(), want), preds
    for src, got in zip(payload, pay):
        assert np.array_equal(got.cpu().numpy(), src[want]), preds
    s = torch.empty(2, dtype=torch.int64, device="cuda")
    tqp.filter_sum_into(dcols, preds, s[:1], s[1:], dcols[0])
    assert tuple(s.tolist()) == oracle.filter_sum(cols, preds, cols[0])[:2], preds


@pytest.mark.parametrize("dt", DTS)
@pytest.mark.parametrize("op", OPS)
def test_literals_at_and_outside_the_type(tqp, dt, op):
    i, wide = np.iinfo(dt), np.iinfo(np.int64)
    n = 4_099
    col = dg.uniform_int(3, 1, n, max(i.min, -(1 << 31)), min(i.max, (1 << 31) - 1), dt)
    col[:6] = [i.min, i.max, 0, -1, i.min + 1, i.max - 1]
    for lit in {i.min, i.max, i.min + 1, i.max - 1, 0, -1, wide.min, wide.max,
                max(i.min - 1, wide.min), min(i.max + 1, wide.max)}:
        check(tqp, [col], [(0, op, int(lit))])
        check(tqp, [col], [(0, op, int(lit)), (0, "!=", 0), (0, ">=", -5), (0, "<=", 100)])


def test_contradictions_and_repeats(tqp):
    col = dg.uniform_int(5, 1, 9_001, -100, 100, np.int8)
    for preds in ([(0, ">", 5), (0, "<", 5)], [(0, "==", 3), (0, "==", 4)], [(0, "==", 3), (0, "!=", 3)],
                  [(0, "!=", 3), (0, "!=", 3), (0, "!=", -7)], [(0, "<", 200)], [(0, "==", 3), (0, "<=", 3)]):
        check(tqp, [col], preds)


@pytest.mark.parametrize("ncols", [1, 2, 3, 4, 5, 8])
def test_columns_loaded_together_and_in_turn(tqp, ncols):
    for n in (1, 7, 8, 9, 2_047, 2_048, 2_049, 30_011):
        cols = [dg.uniform_int(n, c + 1, n, -100, 100, DTS[c % 3]) for c in range(ncols)]
        check(tqp, cols, [(c, OPS[c % 4], 20 - 40 * (c % 2 == 1) * (OPS[c % 4][0] == ">")) for c in range(ncols)],
              payload=cols)


@pytest.mark.parametrize("offset", [1, 3])
@pytest.mark.parametrize("dt", DTS)
def test_columns_at_odd_addresses(tqp, offset, dt):
    n = 20_003
    whole = dg.uniform_int(9, 1, n + offset, -100, 100, dt)
    check(tqp, [whole[offset:]], [(0, ">", -20), (0, "!=", 5)], payload=[whole[offset:]],
          dcols=[dev(whole)[offset:]])


# rows where a block grows from 1 to 2, 4 and 8 tiles of 2048 rows
@pytest.mark.parametrize("n", [(1 << 24) + d for d in (-1, 0, 1)] + [(1 << 25) + 5, (1 << 26) + 4_097])
def test_block_length_changes(tqp, n):
    t = torch.randint(-128, 128, (n,), dtype=torch.int8, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(n))
    for preds, keep in (([(0, "==", 5)], t == 5), ([(0, ">", -100)], t > -100)):
        rows, (p,) = tqp.filter([t], preds, payload=[t])
        want = torch.nonzero(keep).view(-1)
        assert torch.equal(rows.long(), want) and torch.equal(p, t[want])
