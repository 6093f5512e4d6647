"""Programs whose ranges are not sorted and disjoint: a program that shares a
slot with a lower-indexed one is BAD_LAYOUT, by every way the check is made
(owner arrays, a wave's look through the headers; few and many programs, short
and long ones, folded or not), and the order alone costs little."""
import numpy as np
import pytest

from paper_2603_12292_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BAD_LAYOUT = 8


def _api():
    from paper_2603_12292_amd import api
    return api


def _population(N, len_hi, consts_too, seed):
    """Programs in another order than their tokens; some take another's range,
    or its end, or (consts_too) another's constants."""
    rng = np.random.default_rng(seed)
    ps = wl.replicate(wl.random_population(seed, 500, 3, len_hi, 3), (N + 499) // 500)
    perm = rng.permutation(ps.n)[:N]
    off, ln = ps.tok_offset[perm].copy(), ps.tok_len[perm].copy()
    coff, cc = ps.const_offset[perm].copy(), ps.const_count[perm].copy()
    for p in rng.choice(N, size=40, replace=False):
        q = int(rng.integers(N))
        if consts_too and p % 2:
            coff[p], cc[p] = coff[q], max(cc[q], cc[p])
        else:
            off[p], ln[p] = off[q] + ln[q] - 1, max(int(ln[p]) % (len_hi + 1), 3)
    cc = np.minimum(cc, len(ps.consts) - coff).astype(cc.dtype)
    ln = np.minimum(ln, len(ps.tokens) - off).astype(ln.dtype)
    return wl.ProgramSet(ps.tokens, off, ln, ps.consts, coff, cc)


def _shared(off, n):
    """p shares a slot with some q < p (both ranges not empty)."""
    out = np.zeros(len(off), bool)
    for p in range(1, len(off)):
        out[p] = bool(np.any((off[:p] < off[p] + n[p]) & (off[p] < off[:p] + n[:p]) & (n[:p] > 0))) and n[p] > 0
    return out


@pytest.mark.parametrize("N,len_hi", [(64, 70), (70, 12), (300, 90), (4096, 60), (4097, 90), (5000, 16)])
@pytest.mark.parametrize("M", [40, 520])
def test_shared_ranges_are_bad_layout(N, len_hi, M):
    api = _api()
    ps = _population(N, len_hi, True, N + len_hi)
    tok_shared = _shared(ps.tok_offset, ps.tok_len)
    either = tok_shared | _shared(ps.const_offset, ps.const_count)
    assert tok_shared.any() and (either & ~tok_shared).any()
    P = api.DevicePrograms.from_programset(ps)
    X = torch.rand((M, 3), device="cuda") + 1.0
    y = torch.rand((M,), device="cuda")
    thread = api.Context(0)
    thread.set_decoder("thread")
    ref = None
    for c in (None, thread):
        f, st = api.evaluate(P, X, y, "mse", with_status=True, ctx=c)
        st = st.cpu().numpy()
        assert np.array_equal(st == BAD_LAYOUT, tok_shared)
        assert ref is None or np.array_equal(ref, st)
        ref = st
        out = api.evaluate_grad(P, X, y, "mse", with_status=True, ctx=c)
        assert np.array_equal(out[-1].cpu().numpy() == BAD_LAYOUT, either)
    (fb,), (sb,) = api.evaluate_batched([(P, X, y)], "mse", with_status=True)
    assert np.array_equal(sb.cpu().numpy(), ref)
    assert torch.equal(torch.isfinite(fb), torch.isfinite(f))


def test_shared_ranges_with_much_work_folded():
    # (folding: at least FOLD_MIN_CASES cases and FOLD_MIN_WORK program-cases)
    api = _api()
    ps = _population(3000, 70, False, 9)
    P = api.DevicePrograms.from_programset(ps)
    X, y = torch.rand((20000, 3), device="cuda") + 1.0, torch.rand((20000,), device="cuda")
    _, st = api.evaluate(P, X, y, "mse", with_status=True)
    assert np.array_equal(st.cpu().numpy() == BAD_LAYOUT, _shared(ps.tok_offset, ps.tok_len))


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


@pytest.mark.parametrize("call,lo,hi", [("batched", 5, 64), ("evaluate", 66, 120), ("evaluate", 5, 64)])
def test_another_order_costs_little(call, lo, hi):
    # the same 4000 programs; in another order each header is compared with
    # the lower ones, tens of microseconds for a wave
    api = _api()
    N, M = 4000, 1000
    base = wl.replicate(wl.random_population(5, 500, lo, hi, 5), 8)
    perm = np.random.default_rng(1).permutation(N)
    other = wl.ProgramSet(base.tokens, base.tok_offset[perm], base.tok_len[perm], base.consts,
                          base.const_offset[perm], base.const_count[perm])
    X, y = torch.rand((M, 5), device="cuda") + 1.0, torch.rand((M,), device="cuda")
    us = []
    for ps in (base, other):
        P = api.DevicePrograms.from_programset(ps)
        if call == "batched":
            out = [torch.empty(N, dtype=torch.float64, device="cuda")]
            us.append(_us(lambda: api.evaluate_batched([(P, X, y)], "mse", out=out)))
        else:
            us.append(_us(lambda: api.evaluate(P, X, y, "mse")))
    print(f"{call} {lo}..{hi}: sorted {us[0]:.0f} us, in another order {us[1]:.0f} us")
    assert us[1] < us[0] + 150.0
