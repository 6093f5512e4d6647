"""More programs than one launch takes where a program has a wave or a workgroup:
the last programs are served like the first."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _programs(N):
    # one token each: VAR 0, VAR 1, and every 1009th program an invalid VAR 9
    from paper_2603_12292_amd import api, workloads as wl
    i = torch.arange(N, dtype=torch.int64, device="cuda")
    t0, t1, bad = (wl.tok(wl.VAR, v) for v in (0, 1, 9))
    toks = torch.where(i % 2 == 0, t0, t1)
    toks = torch.where(i % 1009 == 0, bad, toks)
    zero = torch.zeros(N, dtype=torch.int64, device="cuda")
    return api.DevicePrograms(toks.to(torch.int16), i, torch.ones(N, dtype=torch.int32, device="cuda"),
                              torch.zeros(1, device="cuda"), zero, zero.to(torch.int32)), i


@pytest.mark.parametrize("N,M", [((1 << 24) + 1018, 120), ((1 << 22) + 1018, 257)])
def test_predictions_of_many_programs(N, M):
    from paper_2603_12292_amd import api
    P, i = _programs(N)
    X = torch.rand((M, 2), device="cuda") + 1.0
    out, st = api.predict(P, X, with_status=True)
    assert torch.equal(st != 0, i % 1009 == 0)
    for k in (0, 1, 2, 1009 * 3, (1 << 22) - 1, 1 << 22, N - 2, N - 1, N // 1009 * 1009):
        if k % 1009 == 0:
            assert bool(torch.isnan(out[k]).all())
        else:
            assert torch.equal(out[k], X[:, k % 2])


def test_folding_more_than_2_24_programs():
    from paper_2603_12292_amd import api
    N, M = (1 << 24) + 1018, 2048
    P, i = _programs(N)
    X = torch.rand((M, 2), device="cuda") + 1.0
    y = torch.rand((M,), device="cuda")
    fit, st = api.evaluate(P, X, y, "mse", with_status=True)
    assert torch.equal(st != 0, i % 1009 == 0)
    want = ((X.double() - y.double()[:, None]) ** 2).mean(0)
    ok = st == 0
    # sums of M squares in float: M * 2^-24 relative at most
    rel = ((fit - want[i % 2]) / want[i % 2]).abs()[ok]
    assert float(rel.max()) < M * 2.0 ** -24
    assert not bool(torch.isfinite(fit[~ok]).any())
