"""Programs that share one large constant table (allowed outside the gradient:
nothing is written by constant): the same results as with tables of their own,
at a cost that does not go by the table's size."""
import numpy as np
import pytest

from paper_2603_12292_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _best(f, n=10):
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


@pytest.mark.parametrize("lo,hi", [(5, 64), (40, 90)])
def test_a_shared_table(lo, hi):
    from paper_2603_12292_amd import api
    N, M, table = 4096, 20_000, 200_000  # (2^26 program-cases and more are folded)
    ps = wl.replicate(wl.random_population(21, 512, lo, hi, 5), 8)
    shared = np.random.default_rng(2).uniform(0.5, 2.0, size=table).astype(np.float32)
    own = np.concatenate([shared[:c] for c in ps.const_count]).astype(np.float32)
    X, y = torch.rand((M, 5), device="cuda") + 1.0, torch.rand((M,), device="cuda")
    P = api.DevicePrograms.from_programset(
        wl.ProgramSet(ps.tokens, ps.tok_offset, ps.tok_len, own, ps.const_offset, ps.const_count))
    Q = api.DevicePrograms.from_programset(
        wl.ProgramSet(ps.tokens, ps.tok_offset, ps.tok_len, shared, np.zeros_like(ps.const_offset),
                      np.full_like(ps.const_count, table)))
    assert torch.equal(api.evaluate(P, X, y).view(torch.int64), api.evaluate(Q, X, y).view(torch.int64))
    a, b = (_best(lambda p=p: api.evaluate(p, X, y)) for p in (P, Q))
    print(f"{lo}..{hi}: own tables {a:.0f} us, one of {table} {b:.0f} us")
    assert b < 1.5 * a
