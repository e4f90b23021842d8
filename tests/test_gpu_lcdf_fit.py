"""Training of the learned CDF's root: the loss before and after some steps against the
same steps with float64 sums, over training sets smaller than a wave, around the
workgroup and full, with even keys, repeated keys and keys beyond a gap; and the
greedy spline knots of the leaves against a plain search through all points."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

H = 32


@pytest.fixture(scope="module")
def tqp():
    import paper_2209_04579_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def sample(kind, n):
    rng = np.random.default_rng(n)
    if kind == "even":
        k = rng.integers(0, 1 << 40, n)
    elif kind == "repeats":
        k = rng.integers(0, 12, n) ** 5 * 1000
    else:
        k = np.where(rng.random(n) < 0.5, rng.integers(0, 1 << 20, n), (1 << 60) + rng.integers(0, 1 << 50, n))
    k[0], k[-1] = 0, k.max() + 1
    return np.sort(k.astype(np.int64))


def f32(a):
    return np.asarray(a).astype(np.float32).astype(np.float64)


def reference(k, steps, lr):
    """Losses seen at each step: sums and gradients in float64, parameters and positions
    on ramps in float32 (repeated keys make ramps narrower than float32 can place)."""
    m, T = len(k), min(len(k), 4096)
    span = float(k[-1] - k[0])
    i = ((np.arange(T) + 0.5) * m / T).astype(np.int64)
    x = ((k[i] - k[0]).astype(np.float64) / span).astype(np.float32).astype(np.float64)
    q = (i + 0.5) / m
    e = (np.arange(H + 1) * (m - 1) / H).astype(np.int64)
    edge = ((k[e] - k[0]).astype(np.float64) / span).astype(np.float32).astype(np.float64)
    s0 = f32(np.maximum(edge[1:] - edge[:-1], 1e-9))
    c0 = f32(0.5 * f32(edge[1:] + edge[:-1]))
    th = f32(np.concatenate([np.zeros(H), np.log(s0), np.full(H, np.log(1.0 / H)), [0.0]]))
    m1, m2, losses = np.zeros(3 * H + 1), np.zeros(3 * H + 1), []
    for step in range(1, steps + 1):
        w, v, c = f32(np.exp(-th[H:2 * H])), np.exp(th[2 * H:3 * H]), f32(c0 + s0 * th[:H])
        z = f32(f32(x[:, None] - c) * w + 0.5)
        h = np.clip(z, 0, 1)
        err = th[-1] + h @ v - q
        losses.append(np.mean(err * err))
        d = 2 * err / T
        act = (z > 0) & (z < 1)
        g = np.concatenate([((d[:, None] * act) * v * -w * s0).sum(0), ((d[:, None] * act) * v * -(z - 0.5)).sum(0),
                            (d[:, None] * v * h).sum(0), [d.sum()]])
        m1, m2 = 0.9 * m1 + 0.1 * g, 0.999 * m2 + 0.001 * g * g
        th = f32(th - lr * (m1 / (1 - 0.9 ** step)) / (np.sqrt(m2 / (1 - 0.999 ** step)) + 1e-12))
        th[H:2 * H] = np.maximum(th[H:2 * H], -40.0)
    return losses


# An error y - q carries 33 roundings of terms below 1 (2e-6), so a loss of errors
# around 0.01 is right to about 4e-4 of itself; losses below that scale to 1e-6.
@pytest.mark.parametrize("kind", ["even", "repeats", "gap"])
@pytest.mark.parametrize("n", [2, 31, 1023, 1025, 4095, 50_000])
def test_losses_match_float64(tqp, kind, n):
    k = sample(kind, n)
    key = torch.from_numpy(k).cuda()
    for steps in (1, 4):
        info = tqp.lcdf_model_info(tqp.lcdf_train([key], sample_stride=1, nleaf=16, steps=steps, lr=1e-3))
        want = reference(k, steps, 1e-3)
        assert info["steps"] == steps
        assert info["loss_first"] == pytest.approx(want[0], rel=2e-3, abs=1e-6)
        assert info["loss_last"] == pytest.approx(want[-1], rel=2e-3, abs=1e-6)
        assert info["loss_best"] == pytest.approx(min(want), rel=2e-3, abs=1e-6)


def test_more_steps_than_the_correction_table(tqp):
    key = torch.from_numpy(sample("even", 5000)).cuda()
    info = tqp.lcdf_model_info(tqp.lcdf_train([key], sample_stride=1, nleaf=16, steps=1030))
    assert info["steps"] == 1030 and info["loss_best"] <= info["loss_first"] and np.isfinite(info["loss_last"])


def spline(kx, kr, key):
    c = int(np.searchsorted(kx, key, side="right"))
    if c == 0 or c == len(kx):
        return kr[0] if c == 0 else kr[-1]
    return kr[c - 1] + (kr[c] - kr[c - 1]) * (float(key - kx[c - 1]) / float(kx[c] - kx[c - 1]))


@pytest.mark.parametrize("kind", ["even", "repeats", "gap"])
@pytest.mark.parametrize("n", [2, 3, 9, 257, 1500])
def test_one_leaf_takes_the_knots_of_a_plain_search(tqp, kind, n):
    k = sample(kind, n)
    raw = tqp.lcdf_train([torch.from_numpy(k).cuda()], sample_stride=1, nleaf=1, steps=0).cpu().numpy()[-96:]
    got_kx, nk = np.frombuffer(raw[:64].tobytes(), np.int64), int(raw[92])
    vals, at, cnt = np.unique(k, return_index=True, return_counts=True)
    run, rs = int(cnt.max()), int(at[cnt.argmax()])
    heavy, kx, kr = run >= 4, [], []
    if not (heavy and rs == 0):
        kx, kr = [int(k[0])], [0.5 / n]
    if heavy:
        kx, kr = kx + [int(k[rs])] * 2, kr + [rs / n, (rs + run) / n]
    if n > 1 and not (heavy and rs + run == n):
        kx, kr = kx + [int(k[-1])], kr + [(n - 0.5) / n]
    while len(kx) < 8:
        err = [0.0 if heavy and rs <= i < rs + run else abs(spline(kx, kr, int(k[i])) - (i + 0.5) / n) for i in range(n)]
        i = int(np.argmax(err))
        if not err[i] > 0:
            break
        kx, kr = map(list, zip(*sorted(zip(kx + [int(k[i])], kr + [(i + 0.5) / n]))))
    assert nk == len(kx) and got_kx[:nk].tolist() == kx
