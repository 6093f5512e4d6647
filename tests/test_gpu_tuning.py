"""The tile-width tuner measures only where the two widths run and differ: a
call whose chunks hold half tiles, a small case set, few program-cases, more
than eight variables or a batch leaves no entry; the widths give the same bits
on every path."""
import numpy as np
import pytest

from paper_2603_12292_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _api():
    from paper_2603_12292_amd import api
    return api


def _problem(N, M, D, seed=1):
    api = _api()
    base = wl.random_population(seed, min(N, 100), 3, 40, D)
    ps = wl.replicate(base, -(-N // base.n))
    if ps.n > N:
        ps = ps.subset(range(N))
    rng = np.random.default_rng(seed)
    X = torch.from_numpy(rng.uniform(0.5, 2.0, size=(M, D)).astype(np.float32)).cuda()
    y = torch.from_numpy(rng.uniform(-1.0, 1.0, size=M).astype(np.float32)).cuda()
    return api.DevicePrograms.from_programset(ps), X, y


def _entries(path):
    if not path.exists():
        return []
    return [ln for ln in path.read_text().splitlines() if not ln.startswith("#")]


@pytest.mark.parametrize("N,M,D,width", [(3000, 512, 3, 4), (300, 500, 3, 4), (6000, 200, 3, 4), (6000, 1000, 3, 8),
                                         (1000, 4096, 3, 8), (300, 70001, 9, 8)])
def test_unmeasured_calls_leave_no_entry(N, M, D, width, tmp_path, monkeypatch):
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("BEAGLE_AUTOTUNE_CACHE", str(path))
    api = _api()
    ctx = api.Context(0)
    P, X, y = _problem(N, M, D)
    api.evaluate(P, X, y, "mse", ctx=ctx)
    assert _entries(path) == []
    assert ctx.tile_width("mse", D, M, P.tokens.numel(), N) == width
    ctx.close()


def test_batch_leaves_no_entry_and_takes_what_is_kept(tmp_path, monkeypatch):
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("BEAGLE_AUTOTUNE_CACHE", str(path))
    api = _api()
    ctx = api.Context(0)
    P, X, y = _problem(300, 70001, 3)
    (f,) = api.evaluate_batched([(P, X, y)], "mse", ctx=ctx)
    assert _entries(path) == []
    g = api.evaluate(P, X, y, "mse", ctx=ctx)      # measures
    assert len(_entries(path)) == 1
    ctx.set_tuning("narrow")
    (h,) = api.evaluate_batched([(P, X, y)], "mse", ctx=ctx)
    for t in (g, h):
        assert np.array_equal(f.cpu().numpy().view(np.uint64), t.cpu().numpy().view(np.uint64))
    ctx.close()


# above the launch that has one width, chunks of whole tiles: streamed rows
# and resident tables, ragged last tiles, up to 16 variables
@pytest.mark.parametrize("N,M,D", [(600, 70001, 9), (600, 70001, 16), (5000, 3001, 9), (5000, 9000, 3), (6000, 700, 9),
                                   (6000, 513, 16), (4097, 255, 2)])
@pytest.mark.parametrize("kind", ["mse", "corr"])
def test_widths_give_the_same_bits(N, M, D, kind):
    api = _api()
    P, X, y = _problem(N, M, D, 7)
    ctx = api.Context(0)
    out = []
    for policy in ("wide", "narrow"):
        ctx.set_tuning(policy)
        out.append(api.evaluate(P, X, y, kind, ctx=ctx).cpu().numpy().view(np.uint64))
        (b,) = api.evaluate_batched([(P, X, y)], kind, ctx=ctx)
        out.append(b.cpu().numpy().view(np.uint64))
    ctx.close()
    for o in out[1:]:
        assert np.array_equal(out[0], o)
