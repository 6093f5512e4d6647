"""Workspaces: what a call is given when memory is short.  Whatever fits the
parts that an evaluation cannot do without fits a context's cap, and a context
without a cap does without the rest when the device has no memory for it."""
import numpy as np
import pytest

from paper_2603_12292_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _api():
    from paper_2603_12292_amd import api
    return api


def _pieces(*sizes):
    return sum((int(s) + 255) // 256 * 256 for s in sizes)


def _chunks(M, N, most, unit):
    C = max(1, -(-M // most))
    if N * C < 4096:
        C = max(C, -(-4096 // N))
    C = min(C, max(1, -(-M // unit)))
    ch = -(-(-(-M // C)) // unit) * unit
    return -(-M // ch)


def _least(ps, M, D, sums, slice_, grad=False):
    """Bytes of the code, the per-token scratch, the lists, the padded cases and
    the partial sums: per token 28, per program 68, cases padded to 2048, at
    least 4096 work items where there are that many pieces of 2048 cases."""
    N, nt, nc = ps.n, max(len(ps.tokens), 1), max(len(ps.consts), 1)
    Mp = -(-M // 2048) * 2048
    C = _chunks(M, N, 32768, 2048)
    G = _chunks(M, N, 1024, 256) if grad else 0
    b = _pieces(*[4 * nt] * 7, 20 * N, 256, 64, 12 * N, 20 * N, 4 * N, 4 * D * Mp, 4 * Mp, 32,
                max(8 * sums * C * slice_, 8 * G * N))
    if grad:
        b += _pieces(4 * nc, 8 * G * nc, 24 * N)
    return b + 256


SHAPES = [(1, 100, 1, 12), (1, 3_000_000, 1, 12), (3, 50_000, 5, 64), (60, 5000, 3, 200), (64, 100_000, 9, 64),
          (1000, 513, 5, 64), (5000, 300, 16, 20), (4096, 20_000, 5, 64)]


def _problem(N, M, D, hi):
    base = wl.random_population(N + D, min(N, 500), 3, hi, D)
    ps = base if base.n == N else wl.replicate(base, -(-N // base.n))
    ps = wl.ProgramSet(ps.tokens, ps.tok_offset[:N], ps.tok_len[:N], ps.consts, ps.const_offset[:N],
                       ps.const_count[:N])
    g = torch.Generator("cuda").manual_seed(N)
    return ps, torch.rand((M, D), device="cuda", generator=g) + 1.0, torch.rand((M,), device="cuda", generator=g)


def _close(a, b):
    # two orders of sums of terms of one sign: within a chunk of at most 32768
    # cases a lane adds a 64th of them in float, then come the lanes
    ok = torch.isfinite(a)
    assert torch.equal(ok, torch.isfinite(b))
    assert bool((a[ok] - b[ok]).abs().le(2 * (32768 // 64 + 64) * 2.0 ** -24 * a[ok].abs()).all())


@pytest.mark.parametrize("N,M,D,hi", SHAPES)
def test_the_least_workspace_is_enough(N, M, D, hi):
    api = _api()
    ps, X, y = _problem(N, M, D, hi)
    P = api.DevicePrograms.from_programset(ps)
    free = api.Context(0)
    f = api.evaluate(P, X, y, "mse", ctx=free)
    _close(f, api.evaluate(P, X, y, "mse", ctx=api.Context(0, _least(ps, M, D, 1, 1))))
    api.evaluate(P, X, y, "corr", ctx=api.Context(0, _least(ps, M, D, 3, 1)))
    if hi <= 64:
        for kind, sums in (("mse", 1), ("corr", 3)):
            api.evaluate_grad(P, X, y, kind, ctx=api.Context(0, _least(ps, M, D, sums, N, grad=True)))
    if N * M <= 1 << 27 and M < 4_000_000:
        a = api.predict(P, X, ctx=free)
        b = api.predict(P, X, ctx=api.Context(0, _least(ps, M, D, 1, 1)))
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(a.nan_to_num(), b.nan_to_num())
    # a batch of the problem twice: the same pieces, a table and a list of work items
    cap = 2 * (_least(ps, M, D, 1, N) - _pieces(256, 64, 4 * N) - 256) + _pieces(2 * 336, 16 * 3 * 8, 128, 512) + 256
    for fb in api.evaluate_batched([(P, X, y)] * 2, "mse", ctx=api.Context(0, cap)):
        _close(f, fb)


def test_extras_are_given_up_when_the_device_is_full():
    api = _api()
    N, M, D = 256, 8_000_000, 16
    ps, X, y = _problem(N, M, D, 30)
    P = api.DevicePrograms.from_programset(ps)
    warm = api.Context(0)
    want = api.evaluate(P, X, y, "mse", ctx=warm)
    need = api.eval_workspace_bytes(P, X, y, "mse")
    bare = 4 * (D + 1) * M
    assert need > 3 * bare  # (derived rows)
    del warm
    torch.cuda.empty_cache()
    keep = bare + bare // 2 + (256 << 20)
    assert keep < need
    held = []
    while torch.cuda.mem_get_info()[0] > keep + (64 << 20):
        held.append(torch.empty(min(torch.cuda.mem_get_info()[0] - keep, 16 << 30), dtype=torch.uint8, device="cuda"))
    full = api.Context(0)
    got = api.evaluate(P, X, y, "mse", ctx=full)
    again = api.evaluate(P, X, y, "mse", ctx=full)
    del held
    torch.cuda.empty_cache()
    assert torch.equal(want, got) and torch.equal(want, again)
