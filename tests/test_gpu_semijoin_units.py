"""GPU parity of the semi-join around the row counts where its workgroups grow (from 256
threads by way of 512 to 1024), with sets that leave smaller workgroups room for them and
sets that do not.  Exact against torch."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kdt", ["int32", "int64"])
@pytest.mark.parametrize("bits", [40, 100_000, 130_000 * 3])
@pytest.mark.parametrize("edge", [1 << 19, 1 << 20, 1 << 21])
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_around_the_sizes(extra, edge, bits, kdt):
    import paper_2209_04579_amd as tqp
    n = edge + extra
    g = torch.Generator(device="cuda").manual_seed(bits + extra)
    sizes = [bits, 90]
    keys = [torch.randint(-2, z + 2, (n,), device="cuda", generator=g).to(getattr(torch, kdt)) for z in sizes]
    sets, member = [], []
    for z in sizes:
        m = torch.randperm(z, device="cuda", generator=g)[: 1 + z // 2]
        b = torch.empty(tqp.keyset_words(z), dtype=torch.int32, device="cuda")
        tqp.keyset_build_into(m, 0, z, b)
        sets.append((b, 0, z))
        has = torch.zeros(z + 4, dtype=torch.bool, device="cuda")
        has[m + 2] = True
        member.append(has)
    rows = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    kout = [torch.zeros_like(k) for k in keys]
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    ws = tqp.workspace(tqp.semijoin_workspace_bytes(n, keys[0].dtype))
    tqp.semijoin_into(keys, sets, rows, cnt, ws, keys_out=kout)
    want = torch.nonzero(member[0][keys[0].long() + 2] & member[1][keys[1].long() + 2]).flatten()
    m = int(cnt.item())
    assert m == want.numel() and torch.equal(rows[:m], want.int())
    for src, got in zip(keys, kout):
        assert torch.equal(got[:m], src[want])
