"""Work lists long enough to be handed out by the shared counters: every item
is done once (copies of a program agree bit for bit, and with a short list
that is walked without counters), and handing them out does not decide the
time of a call."""
import numpy as np
import pytest

from paper_2603_12292_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _api():
    from paper_2603_12292_amd import api
    return api


def _data(M, D, seed=3):
    rng = np.random.default_rng(seed)
    X = rng.uniform(0.5, 2.0, size=(M, D)).astype(np.float32)
    y = rng.uniform(-1.0, 1.0, size=M).astype(np.float32)
    return torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()


def _bits(t):
    return t.cpu().numpy().view(np.uint64)


# (copies of 100 programs, cases): a resident table of one and of several
# tiles, streamed rows in one chunk and in several, both claimed
@pytest.mark.parametrize("copies,M", [(500, 300), (500, 1300), (300, 6000), (50, 60000)])
@pytest.mark.parametrize("kind", ["mse", "corr"])
def test_copies_agree(copies, M, kind):
    api = _api()
    base = wl.random_population(5, 100, 3, 40, 3)
    X, y = _data(M, 3)
    one = _bits(api.evaluate(api.DevicePrograms.from_programset(base), X, y, kind))
    many = _bits(api.evaluate(api.DevicePrograms.from_programset(wl.replicate(base, copies)), X, y, kind))
    many = many.reshape(copies, -1)
    assert np.array_equal(many, np.broadcast_to(many[0], many.shape))
    a, b = one.view(np.float64), many[0].copy().view(np.float64)
    assert np.array_equal(np.isfinite(a), np.isfinite(b))
    ok = np.isfinite(a)
    # other chunks: the binary64 sums' rounding, amplified by 1 - r^2's cancellation
    assert np.all(np.abs(a[ok] - b[ok]) <= 1e-9 * np.maximum(1.0, np.abs(a[ok])))


def test_gradient_copies_agree():
    api = _api()
    base = wl.random_population(6, 100, 8, 40, 3)
    X, y = _data(700, 3)
    P = api.DevicePrograms.from_programset(wl.replicate(base, 400))
    f, g = api.evaluate_grad(P, X, y, "mse")
    f = _bits(f).reshape(400, -1)
    g = g.cpu().numpy().view(np.uint32).reshape(400, -1)
    assert np.array_equal(f, np.broadcast_to(f[0], f.shape))
    assert np.array_equal(g, np.broadcast_to(g[0], g.shape))


def test_batch_copies_agree():
    api = _api()
    base = wl.random_population(7, 100, 3, 40, 3)
    probs = [(api.DevicePrograms.from_programset(wl.replicate(base, c)), *_data(M, 3, M)) for c, M in
             ((60, 900), (1, 50), (80, 5000), (3, 30000))]
    for (P, X, y), f in zip(probs, api.evaluate_batched(probs, "corr")):
        assert np.array_equal(_bits(f), _bits(api.evaluate(P, X, y, "corr")))


def _us(f, n=20):
    f(), f()
    best = 1e9
    for _ in range(5):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(n):
            f()
        t1.record()
        torch.cuda.synchronize()
        best = min(best, t0.elapsed_time(t1) / n * 1e3)
    return best


def test_many_short_items_cost_what_few_long_ones_do():
    """The same programs x cases as 100 000 x 256 and as 6250 x 4096: the
    gradient's items are the same in size (one chunk of 256 cases, or 16), but
    the lists of the first are 16 times as long per case."""
    api = _api()
    base = wl.random_population(8, 250, 8, 40, 3)
    many = api.DevicePrograms.from_programset(wl.replicate(base, 400))
    few = api.DevicePrograms.from_programset(wl.replicate(base, 25))
    Xs, ys = _data(256, 3)
    Xl, yl = _data(4096, 3)
    a = _us(lambda: api.evaluate_grad(many, Xs, ys, "mse"))
    b = _us(lambda: api.evaluate_grad(few, Xl, yl, "mse"))
    c = _us(lambda: api.evaluate(many, Xs, ys, "mse"))
    print(f"100000 x 256: {a:.0f} us, 6250 x 4096: {b:.0f} us, without gradients {c:.0f} us")
    assert a < 2.2 * b
