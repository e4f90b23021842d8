"""GPU parity of the semi-join where the device chooses between two kernels and a single
pass: around the size where the choice begins (200 MB of keys), around whole tiles of the single pass
(6144 int64 rows, 12288 int32 rows), for sets that keep few and many rows, and in parts,
with payloads, unaligned columns and a set that is not staged.  Exact against torch."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PART = 1 << 25


def _first(ns, kdt):
    """The fewest rows of ns key columns above 200 MB."""
    return 200_000_000 // (ns * (4 if kdt == "int32" else 8)) + 1


def _tiled(ns, kdt):
    return -(-_first(ns, kdt) // 12288) * 12288


def _run(n, ns, kdt, share, noalloc=False, unaligned=False, big=False, replay=False):
    import paper_2209_04579_amd as tqp
    g = torch.Generator(device="cuda").manual_seed(n % 1000 + ns)
    sizes = [100_000, 25, 1000, 3000][:ns]
    if big:
        sizes[1] = 3_000_000
    kept = [max(1, int(z * share ** (1 / ns))) for z in sizes]
    keys = []
    for z in sizes:
        k = torch.randint(-1, z + 2, (n + 1,), device="cuda", generator=g).to(getattr(torch, kdt))
        keys.append(k[1:] if unaligned else k[:n].clone())
    sets = []
    for z, m in zip(sizes, kept):
        bits = torch.empty(tqp.keyset_words(z), dtype=torch.int32, device="cuda")
        tqp.keyset_build_into(torch.arange(0, m, device="cuda"), 0, z, bits)
        sets.append((bits, 0, z))
    pay = [torch.randint(-100, 100, (n,), device="cuda", generator=g).to(torch.int8),
           torch.randint(-(1 << 40), 1 << 40, (n,), device="cuda", generator=g)]
    pout = [torch.zeros_like(p) for p in pay]
    rows = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    kout = [torch.zeros_like(k) for k in keys]
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    ws = None if noalloc else tqp.workspace(tqp.semijoin_workspace_bytes(n, keys[0].dtype))

    def call():
        if noalloc:
            tqp.semijoin_noalloc_into(keys, sets, rows, cnt, keys_out=kout, payload_in=pay, payload_out=pout)
        else:
            tqp.semijoin_into(keys, sets, rows, cnt, ws, keys_out=kout, payload_in=pay, payload_out=pout)

    def check():
        want = torch.nonzero(torch.stack([(k >= 0) & (k < m) for k, m in zip(keys, kept)]).all(0)).flatten()
        m = int(cnt.item())
        assert m == want.numel() and torch.equal(rows[:m], want.int())
        assert m == n or int(rows[m].item()) == -7 or replay
        for src, got in zip(keys + pay, kout + pout):
            assert torch.equal(got[:m], src[want])

    call()
    check()
    if replay:
        # replays see new sets: the choice is made again on each
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                call()
        for share in (0.01, 0.8, 0.01):
            kept = [max(1, int(z * share ** (1 / ns))) for z in sizes]
            for (bits, lo, z), m in zip(sets, kept):
                tqp.keyset_build_into(torch.arange(0, m, device="cuda"), lo, z, bits)
            graph.replay()
            torch.cuda.synchronize()
            check()


@pytest.mark.parametrize("kdt", ["int32", "int64"])
@pytest.mark.parametrize("at", ["below", "first", -1, 0, 1])
@pytest.mark.parametrize("share", [0.02, 0.7, 1.0])
def test_around_whole_tiles(at, share, kdt):
    first = _first(3, kdt)
    _run({"below": first - 1, "first": first}.get(at) or _tiled(3, kdt) + at, 3, kdt, share)


@pytest.mark.parametrize("kdt", ["int32", "int64"])
@pytest.mark.parametrize("form,ns", [(f, ns) for f in ("plain", "unaligned", "noalloc") for ns in (1, 2, 4)]
                         + [("big", 2), ("big", 4)])
def test_forms(form, ns, kdt):
    _run(_tiled(ns, kdt) + 777, ns, kdt, 0.6, noalloc=form == "noalloc", unaligned=form == "unaligned", big=form == "big")


@pytest.mark.parametrize("kdt", ["int32", "int64"])
@pytest.mark.parametrize("share", [0.02, 0.6])
@pytest.mark.parametrize("rest", [5, 17_000_005])
def test_parts(rest, share, kdt):
    _run(PART + rest, 3, kdt, share, noalloc=True)


@pytest.mark.parametrize("noalloc", [False, True])
def test_replays_choose_again(noalloc):
    _run(_tiled(3, "int64") + 5, 3, "int64", 0.7, noalloc=noalloc, replay=True)
