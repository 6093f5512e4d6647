"""Case chunks: sums over many chunks match the outputs, batches cut their
problems as single calls do, and the split of a few programs' cases keeps the
chip busy."""
import math

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
    y = (X[:, 0] * X[:, -1] + rng.uniform(-1.0, 1.0, size=M)).astype(np.float32)
    return X, y, torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()


# programs and cases: few and many chunks (to either side of where a wave adds
# the partial sums), ragged last tiles, a multiple of the programs in a round
@pytest.mark.parametrize("N,M", [(7, 3000), (7, 5000), (24, 60001), (96, 20000), (3, 300001), (1500, 9000), (1700, 9000)])
def test_sums_over_chunks_match_the_outputs(N, M):
    api = _api()
    ps = wl.random_population(17, N, 3, 30, 2)
    X, y, Xd, yd = _data(M, 2)
    P = api.DevicePrograms.from_programset(ps)
    idx = list(range(N)) if N * M < 1 << 22 else list(range(0, N, N // 12))
    out = api.predict(api.DevicePrograms.from_programset(ps.subset(idx)), Xd).cpu().numpy().astype(np.float64)
    mse = api.evaluate(P, Xd, yd, "mse").cpu().numpy()[idx]
    corr = api.evaluate(P, Xd, yd, "corr").cpu().numpy()[idx]
    r4 = api.evaluate_score(P, Xd, yd, "r4", 1000.0).cpu().numpy()[idx]
    t = y.astype(np.float64)
    w = t - t.mean()
    for o, f, c, s in zip(out, mse, corr, r4):
        if not np.all(np.isfinite(o)) or np.abs(o).max() > 1e6:
            continue
        # the rounding of M binary64 additions of non-negative terms
        ref = math.fsum((o - t) ** 2) / M
        assert abs(f - ref) <= (M + 64) * 2.0 ** -52 * ref
        u = o - o[0]
        sxx = math.fsum(u * u) - math.fsum(u) ** 2 / M
        if not sxx > 1e-6 * math.fsum(u * u):
            continue
        sxy = math.fsum(u * w) - math.fsum(u) * math.fsum(w) / M
        r = sxy / math.sqrt(sxx * math.fsum(w * w))
        # sums of M terms each, amplified by at most 1e6 in sxx
        tol = 4e6 * (M + 64) * 2.0 ** -52
        assert abs(c - (1 - r * r)) <= tol
        assert abs(s - 1000.0 * r ** 4 * M) <= 2000.0 * M * tol


@pytest.mark.parametrize("kind", ["mse", "corr"])
def test_batch_of_many_and_few_chunks_equals_single(kind):
    api = _api()
    probs = []
    for q, (N, M) in enumerate([(3, 40000), (24, 50000), (300, 700), (1500, 4100), (5, 4000), (96, 9001)]):
        _, _, Xd, yd = _data(M, 1 + q, q)
        probs.append((api.DevicePrograms.from_programset(wl.random_population(q, N, 3, 40, 1 + q)), Xd, yd))
    for (P, X, y), f in zip(probs, api.evaluate_batched(probs, kind)):
        one = api.evaluate(P, X, y, kind)
        assert np.array_equal(one.cpu().numpy().view(np.uint64), f.cpu().numpy().view(np.uint64))


def _us(f, n=20):
    f(), f(), f()
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


# the same programs x cases with fewer programs: fewer work items unless the
# cases are cut finer
@pytest.mark.parametrize("few,many", [((4096, 4096), (16384, 1024)), ((100, 100000), (1000, 10000))])
def test_few_programs_fill_the_chip(few, many):
    api = _api()
    t = []
    for N, M in (few, many):
        ps = wl.replicate(wl.random_population(9, 100, 5, 64, 5), -(-N // 100)).subset(range(N))
        _, _, X, y = _data(M, 5)
        P = api.DevicePrograms.from_programset(ps)
        ctx = api.Context(0)
        ctx.set_tuning("wide")
        t.append(_us(lambda: api.evaluate(P, X, y, "mse", ctx=ctx)))
        ctx.close()
    print(f"{few}: {t[0]:.0f} us, {many}: {t[1]:.0f} us")
    assert t[0] < 1.5 * t[1]
