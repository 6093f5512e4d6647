"""Staged input rows on the GPU: rows holding a base unary operator of a
variable, the evaluator's stream of rows and its resident table give the
outputs and sums that plain evaluation gives."""
import math

import numpy as np
import pytest

from paper_2603_12292_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

T = wl.tok


def _api():
    from paper_2603_12292_amd import api
    return api


def _programs(D, seed):
    """Random programs, every base unary operator of every variable as a push
    and as the operand of a fused pair on either side, operator runs on a
    variable, 64 and 65 and 200 VAR words, register needs 5 and 9."""
    rng = np.random.default_rng(seed)
    progs = [wl.random_program(rng, int(rng.integers(1, 65)), D) for _ in range(20)]
    for d in range(D):
        for u in wl.UNARY_OPS:
            progs.append(([T(wl.VAR, d), T(u)], []))
            progs.append(([T(wl.CONST, 0), T(wl.VAR, d), T(u), T(wl.SUB)], [1.5]))
            progs.append(([T(wl.VAR, d), T(u), T(wl.CONST, 0), T(wl.DIV)], [0.75]))
    progs.append(([T(wl.VAR, 0)] + [T(wl.SQRT), T(wl.SIN), T(wl.COS)] * 10, []))
    for k in (63, 64, 65, 200):
        toks = [T(wl.VAR, 0)]
        for j in range(k - 1):
            toks += [T(wl.VAR, j % D)] + ([T(wl.SIN)] if j % 3 == 0 else []) + [T(wl.ADD)]
        progs.append((toks, []))

    def tree(n):
        if n == 1:
            return [T(wl.VAR, n % D)]
        return tree(n - 1) + tree(n - 1) + [T(wl.ADD)]

    progs += [(tree(5), []), (tree(9), [])]
    return progs


@pytest.mark.parametrize("D", [1, 5, 16])
def test_derived_rows_change_no_output(D):
    # 16 programs and more stage the derived rows, fewer do not
    api = _api()
    progs = _programs(D, 31 + D)
    rng = np.random.default_rng(D)
    X = rng.uniform(-4, 4, size=(600, D)).astype(np.float32)
    X[:8, 0] = [0.0, -0.0, 1e-40, np.inf, -np.inf, np.nan, 3e38, 81.0]
    Xd = torch.from_numpy(X).cuda()
    run = lambda ps: api.predict(api.DevicePrograms.from_programset(wl.pack_programs(ps)), Xd).cpu().numpy()
    whole = run(progs)
    parts = np.concatenate([run(progs[i:i + 12]) for i in range(0, len(progs), 12)])
    assert np.array_equal(np.isnan(whole), np.isnan(parts))
    ok = ~np.isnan(whole)
    assert np.array_equal(whole.view(np.uint32)[ok], parts.view(np.uint32)[ok])


@pytest.mark.parametrize("tuning", ["wide", "narrow"])
@pytest.mark.parametrize("copies", [1, 50])
@pytest.mark.parametrize("M", [1, 255, 256, 257, 511, 513, 1025, 4097, 9000])
def test_sums_match_the_outputs(M, copies, tuning):
    # one copy: the stream of rows, chunks of half and whole tiles; 50 copies
    # (over 4096 programs): also the resident table where M allows it.  The
    # tolerance is the rounding of M binary64 additions of non-negative terms.
    api = _api()
    progs = _programs(4, 7)
    rng = np.random.default_rng(M)
    X = rng.uniform(0.5, 2.0, size=(M, 4)).astype(np.float32)
    y = rng.uniform(-1.0, 1.0, size=M).astype(np.float32)
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    out = api.predict(api.DevicePrograms.from_programset(wl.pack_programs(progs)), Xd).cpu().numpy().astype(np.float64)
    with np.errstate(over="ignore", invalid="ignore"):
        ref = [math.fsum((o - y.astype(np.float64)) ** 2) / M if np.all(np.isfinite(o)) else np.nan for o in out]
    ctx = api.Context(0)
    ctx.set_tuning(tuning)
    ps = wl.replicate(wl.pack_programs(progs), copies)
    assert copies == 1 or ps.n >= 4096
    fit = api.evaluate(api.DevicePrograms.from_programset(ps), Xd, yd, "mse", ctx=ctx).cpu().numpy()
    assert np.array_equal(fit.reshape(copies, -1).view(np.uint64),
                          np.broadcast_to(fit[:len(progs)], (copies, len(progs))).copy().view(np.uint64))
    for p, r in enumerate(ref):
        if math.isfinite(r):
            assert abs(fit[p] - r) <= (M + 64) * 2.0 ** -52 * r, (p, fit[p], r)
