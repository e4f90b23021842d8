"""GPU parity of the semi-join scan on tables, and on last parts of a table taken in
parts, around one chunk of 512 rows: shorter ones load key by key, longer ones whole
chunks.  Exact against torch."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PART = 1 << 25


@pytest.mark.parametrize("kdt", ["int32", "int64"])
@pytest.mark.parametrize("ns", [1, 3])
@pytest.mark.parametrize("n,noalloc", [(n, na) for n in (1, 7, 511, 512, 513, 1025) for na in (False, True)]
                         + [(PART + r, True) for r in (1, 511, 512, 513)])
def test_around_one_chunk(n, noalloc, ns, kdt):
    import paper_2209_04579_amd as tqp
    g = torch.Generator(device="cuda").manual_seed(n % 1000 + ns)
    keys = [torch.randint(0, 90, (n,), device="cuda", generator=g).to(getattr(torch, kdt)) for _ in range(ns)]
    for k in keys:
        k[-1] = 3
    bits = torch.empty(tqp.keyset_words(90), dtype=torch.int32, device="cuda")
    tqp.keyset_build_into(torch.arange(0, 45, device="cuda"), 0, 90, bits)
    rows = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    kout = [torch.zeros_like(k) for k in keys]
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    sets = [(bits, 0, 90)] * ns
    if noalloc:
        tqp.semijoin_noalloc_into(keys, sets, rows, cnt, keys_out=kout)
    else:
        ws = tqp.workspace(tqp.semijoin_workspace_bytes(n, keys[0].dtype))
        tqp.semijoin_into(keys, sets, rows, cnt, ws, keys_out=kout)
    want = torch.nonzero(torch.stack([k < 45 for k in keys]).all(0)).flatten()
    m = int(cnt.item())
    assert m == want.numel() and torch.equal(rows[:m], want.int())
    for src, got in zip(keys, kout):
        assert torch.equal(got[:m], src[want])
