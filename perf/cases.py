"""Performance cases of the library: what a user's program asks of it.

Every case is one call of the Python API (paper_2603_12292_amd.api) on inputs
that the program holds on the GPU: a population of postfix programs in the
packed layout (or in fixed-capacity slots, as the generation step writes
them), fitness cases X and targets y.  Sizes come from the repository's own
workloads (plain-tiny, plain-mid, the paper's regime, the generation loop, the
ragged batch, the adjoint) and from the ranges around them.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs on the GPU, made from the seed alone
    run(state)          one call, its whole outputs
    work(case)          bytes and operations that the call cannot do without
    exact(case, seed)   the same outputs in binary64, by plain torch
"""
import math

import torch

from paper_2603_12292_amd import api

# Token format of the library's input: opcode | arg << 8.
ADD, SUB, MUL, DIV, SIN, COS, EXP, LOG, SQRT, VAR, CONST = range(11)
SQUARE, RECIP, TAN, ASIN, ACOS, ATAN, TANH = range(11, 18)
UNARY_9 = (SIN, COS, EXP, LOG, SQRT)
UNARY_16 = UNARY_9 + (SQUARE, RECIP, TAN, ASIN, ACOS, ATAN, TANH)
MAX_CONSTS = 8
MAX_SCORE = 1000.0
DEVICE = "cuda:0"


def listed():
    return [
        # a first look at a small problem, called interactively: latency and
        # the number of launches decide (the plain-tiny workload)
        dict(name="eval_tiny_mse", call="evaluate", kind="mse", N=256, M=1000, D=3, lo=3, hi=32, ops=9),
        # the paper's Eq. 2 score of a small population on an odd number of
        # cases, a quarter of the targets undefined
        dict(name="score_small_r4", call="score", kind="r4", N=1000, M=777, D=4, lo=5, hi=64, ops=9),
        # the benchmark workload (plain-mid): one generation's evaluation
        dict(name="eval_mid_corr", call="evaluate", kind="corr", N=4096, M=100_000, D=5, lo=5, hi=64, ops=9),
        # the generation loop's data (D = 9, 10^6 cases), programs grown past
        # 64 tokens
        dict(name="eval_wide_mse", call="evaluate", kind="mse", N=2048, M=1_000_000, D=9, lo=5, hi=96, ops=9),
        # the paper's regime: about 10^6 individuals on 512 cases
        dict(name="eval_paper_corr", call="evaluate", kind="corr", N=1 << 20, M=512, D=5, lo=5, hi=64, ops=9),
        # the paper's whole operator table, at the population size its
        # schedule ends with
        dict(name="eval_ops16_mse", call="evaluate", kind="mse", N=250_000, M=512, D=5, lo=3, hi=32, ops=16),
        # outputs of the best individuals on a validation set
        dict(name="predict_best", call="predict", N=100, M=100_000, D=5, lo=5, hi=64, ops=9),
        # one gradient step of constant tuning over a whole population (the
        # adjoint workload)
        dict(name="grad_mid_mse", call="grad", kind="mse", N=4096, M=100_000, D=5, lo=8, hi=64, ops=9),
        # constant tuning of a few hundred survivors under the correlation
        # fitness, odd sizes
        dict(name="grad_small_corr", call="grad", kind="corr", N=301, M=4999, D=3, lo=8, hi=64, ops=9),
        # many independent problems of unlike sizes in one call
        dict(name="batched_ragged", call="batched", kind="corr", problems=24, N=512, m_lo=1000, m_hi=300_000, lo=5,
             hi=96, ops=9),
        # the generation loop's variation: tournaments, crossover, mutation
        dict(name="generation_tournament", call="generation", N=16384, D=9, lo=5, hi=96, max_len=128, ops=9),
        # the paper's own variation: microcosm selection, mutation only
        dict(name="generation_microcosm", call="microcosm", N=1_000_000, D=5, lo=3, hi=40, max_len=64, ops=9),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(("evaluate", "evaluate", "evaluate", "score", "predict", "grad", "batched", "generation",
                       "microcosm"))
    lo, hi = rng.choice(((3, 32), (5, 64), (5, 96)))
    D = rng.randint(1, 9)
    ops = rng.choice((9, 9, 9, 16))
    if call == "generation":
        return dict(call=call, N=_log(rng, 100, 60_000), D=D, lo=lo, hi=hi, max_len=rng.choice((100, 128, 200)), ops=ops)
    if call == "microcosm":
        return dict(call=call, N=_log(rng, 1000, 2_000_000), D=D, lo=3, hi=rng.randint(8, 56), max_len=64, ops=ops)
    if call == "batched":
        return dict(call=call, kind=rng.choice(("mse", "corr")), problems=rng.randint(2, 32), N=_log(rng, 32, 700),
                    m_lo=_log(rng, 100, 3000), m_hi=_log(rng, 5000, 200_000), lo=lo, hi=hi, ops=9)
    # programs x cases within the largest listed case of the call
    top = {"evaluate": 1 << 30, "score": 1 << 29, "predict": 1 << 25, "grad": 1 << 28}[call]
    n_hi = {"evaluate": 1 << 20, "score": 1 << 20, "predict": 1000, "grad": 20_000}[call]
    N = _log(rng, 32, n_hi)
    M = _log(rng, 64, min(1_000_000, max(128, top // N)))
    case = dict(call=call, N=N, M=M, D=D, lo=max(lo, 8) if call == "grad" else lo, hi=hi, ops=ops)
    if call != "predict":
        case["kind"] = rng.choice(("r4", "point") if call == "score" else ("mse", "corr"))
    return case


# ---- inputs -----------------------------------------------------------------

def _slots(g, N, lo, hi, D, ops, consts=True):
    """N random postfix programs of lengths U{lo..hi} as token slots [N, hi]
    (int64, -1 past the end), their lengths and their constant counts: each
    token uniform over the symbols that still let the program close."""
    unary = torch.tensor(UNARY_9 if ops == 9 else UNARY_16, device=DEVICE)
    n_un = unary.numel()
    n_term = D + (1 if consts else 0)
    L = torch.randint(lo, hi + 1, (N,), generator=g, device=DEVICE)
    tok = torch.full((N, hi), -1, dtype=torch.int64, device=DEVICE)
    depth = torch.zeros(N, dtype=torch.int64, device=DEVICE)
    nc = torch.zeros(N, dtype=torch.int64, device=DEVICE)
    for pos in range(hi):
        r = L - pos - 1
        live = r >= 0
        k_t = torch.where(depth <= r, n_term, 0)
        k_u = torch.where((depth >= 1) & (depth - 1 <= r), n_un, 0)
        k_b = torch.where((depth >= 2) & (depth - 2 <= r), 4, 0)
        u = torch.rand(N, generator=g, device=DEVICE, dtype=torch.float64)
        k = (u * (k_t + k_u + k_b)).long()
        term = k < k_t
        un = ~term & (k < k_t + k_u)
        cst = term & (k == D) & (nc < MAX_CONSTS) & live
        var = torch.where(k < D, k, 0)
        t = torch.where(cst, CONST | (nc << 8), VAR | (var << 8))
        t = torch.where(un, unary[(k - k_t).clamp(0, n_un - 1)], t)
        t = torch.where(~term & ~un, k - k_t - k_u, t)
        tok[:, pos] = torch.where(live, t, -1)
        nc += cst
        depth += torch.where(live, torch.where(term, 1, torch.where(un, 0, -1)), 0)
    return tok, L, nc


def _place_constants(g, tok):
    """1..8 of every program's terminals become constants, in token order."""
    is_term = ((tok & 0xFF) == VAR) & (tok >= 0)
    key = torch.where(is_term, torch.rand(tok.shape, generator=g, device=DEVICE), 2.0)
    rank = key.argsort(1).argsort(1)
    k = torch.minimum(torch.randint(1, MAX_CONSTS + 1, (tok.shape[0],), generator=g, device=DEVICE), is_term.sum(1))
    pick = is_term & (rank < k[:, None])
    slot = pick.long().cumsum(1) - 1
    return torch.where(pick, CONST | (slot << 8), tok), k


def _packed(g, tok, L, nc):
    """The library's packed layout of token slots, constants U(-5, 5) in one
    table row of MAX_CONSTS per program."""
    tok_offset = L.cumsum(0) - L
    const_offset = torch.arange(L.numel(), device=DEVICE) * MAX_CONSTS
    consts = torch.rand(L.numel() * MAX_CONSTS, generator=g, device=DEVICE) * 10 - 5
    return api.DevicePrograms(tok[tok >= 0].to(torch.int16), tok_offset, L.int(), consts, const_offset, nc.int())


def _data(g, M, D, undefined=False):
    """X ~ U(1, 10) (U(1, 5) with undefined targets), y a smooth function of a
    few variables with 1 % noise, or log(x0 - 2)(1 + x1 / 4): NaN on a
    quarter of the domain."""
    X = torch.rand((M, D), generator=g, device=DEVICE) * (4 if undefined else 9) + 1
    v = X.double()
    c = torch.rand(4, generator=g, device=DEVICE, dtype=torch.float64) * 4 - 2
    x0, x1, x2 = v[:, 0], v[:, 1 % D], v[:, 2 % D]
    if undefined:
        y = torch.log(x0 - 2) * (1 + x1 / 4)
    else:
        y = c[0] * x0 * torch.sin(x1) + c[1] * torch.log(x2) + c[2] * torch.sqrt(x0 * x2) + c[3]
        y = y + 0.01 * y.square().mean().sqrt() * torch.randn(M, generator=g, device=DEVICE, dtype=torch.float64)
    return X, y.float()


def _population(g, case, D, consts=True):
    tok, L, nc = _slots(g, case["N"], case["lo"], case["hi"], D, case["ops"], consts)
    if not consts:
        tok, nc = _place_constants(g, tok)
    return tok, L, nc


def _inputs(case, seed):
    """Everything of a case that follows from its seed: token slots beside the
    library's own inputs."""
    g = torch.Generator(DEVICE).manual_seed(seed * 1_000_003 + 17)
    call = case["call"]
    if call == "batched":
        out = []
        for _ in range(case["problems"]):
            D, e = (torch.rand(2, generator=g, device=DEVICE, dtype=torch.float64)).tolist()
            D = 1 + int(D * 9)
            M = int(round(math.exp(math.log(case["m_lo"]) + e * math.log(case["m_hi"] / case["m_lo"]))))
            tok, L, nc = _population(g, case, D)
            progs = _packed(g, tok, L, nc)
            out.append((tok, progs, *_data(g, M, D)))
        return out
    D = case["D"]
    tok, L, nc = _population(g, case, D, consts=call != "grad")
    if call in ("generation", "microcosm"):
        N, max_len = case["N"], case["max_len"]
        slots = torch.zeros((N, max_len), dtype=torch.int16, device=DEVICE)
        slots[:, :case["hi"]] = tok.clamp(min=0).to(torch.int16)
        consts = torch.rand((N, MAX_CONSTS), generator=g, device=DEVICE) * 10 - 5
        consts = torch.where(torch.arange(MAX_CONSTS, device=DEVICE) < nc[:, None], consts, 0.0)
        progs = api.DevicePrograms.from_fixed(slots, L.int(), consts, nc.int())
        fit = torch.rand(N, generator=g, device=DEVICE, dtype=torch.float64)
        fit[torch.rand(N, generator=g, device=DEVICE) < 0.01] = float("nan")
        return progs, fit
    progs = _packed(g, tok, L, nc)
    return (tok, progs, *_data(g, case["M"], D, undefined=call == "score"))


def prepare(case, seed):
    call = case["call"]
    inp = _inputs(case, seed)
    if call == "batched":
        problems = [(p, X, y) for _, p, X, y in inp]
        # results land in arrays that the program keeps
        out = [torch.empty(p.n, dtype=torch.float64, device=DEVICE) for p, _, _ in problems]
        return dict(case=case, problems=problems, out=out)
    if call in ("generation", "microcosm"):
        progs, fit = inp
        mutate = call == "microcosm"
        params = api.GenParams(tournament=1 if mutate else 4, p_crossover=0.0 if mutate else 0.9,
                               p_mutation=1.0 if mutate else 0.1, max_len=case["max_len"], max_consts=MAX_CONSTS,
                               op_set=1 if case["ops"] == 16 else 0)
        spare = api.Slots.empty(case["N"], case["max_len"], MAX_CONSTS, DEVICE)
        return dict(case=case, progs=progs, fit=fit, params=params, spare=spare, seed=seed)
    _, progs, X, y = inp
    return dict(case=case, progs=progs, X=X, y=y)


def run(state):
    case = state["case"]
    call = case["call"]
    if call == "evaluate":
        return api.evaluate(state["progs"], state["X"], state["y"], case["kind"])
    if call == "score":
        return api.evaluate_score(state["progs"], state["X"], state["y"], case["kind"], MAX_SCORE)
    if call == "predict":
        return api.predict(state["progs"], state["X"])
    if call == "grad":
        return api.evaluate_grad(state["progs"], state["X"], state["y"], case["kind"])
    if call == "batched":
        return api.evaluate_batched(state["problems"], case["kind"], out=state["out"])
    if call == "generation":
        s = api.generation(state["progs"], state["fit"], state["params"], case["D"], state["seed"], 1,
                           out=state["spare"])
        return s.tokens, s.len, s.consts, s.const_count
    s, tau, n = api.generation_microcosm(state["progs"], state["fit"], state["params"], case["D"], state["seed"], 1,
                                         case["N"], out=state["spare"], with_selection=True)
    return s.tokens, s.len, s.consts, s.const_count, tau, n


def work(case):
    """Inputs read once, outputs written once; one operation per operator
    application and case (0.63 of the tokens are operators), the fitness terms
    on top; a gradient twice that again."""
    call, N = case["call"], case["N"]
    mean = (case["lo"] + case["hi"]) / 2
    if call in ("generation", "microcosm"):
        child = case["max_len"] * 2 + MAX_CONSTS * 4 + 8
        parents = 2 if call == "generation" else 1
        return dict(bytes=N * (8 + parents * (mean * 2 + MAX_CONSTS * 2 + 8) + child), flops=0)
    programs = N * (mean * 2 + 24 + 4 * 4)
    if call == "batched":
        mean_m = (case["m_hi"] - case["m_lo"]) / math.log(case["m_hi"] / case["m_lo"])
        q = case["problems"]
        return dict(bytes=q * (programs + mean_m * 24 + N * 8), flops=q * N * mean_m * (0.63 * mean + 3))
    M, D = case["M"], case["D"]
    io = programs + M * (D + 1) * 4
    ops = N * M * 0.63 * mean
    if call == "predict":
        return dict(bytes=io + N * M * 4, flops=ops)
    flops = ops + N * M * (3 if case["kind"] in ("mse", "point") else 5)
    if call == "grad":
        return dict(bytes=io + N * (8 + 4 * 4), flops=3 * flops)
    return dict(bytes=io + N * 8, flops=flops)


# ---- binary64 values --------------------------------------------------------

def _unary64(op, x):
    if op == SIN:
        return torch.sin(x)
    if op == COS:
        return torch.cos(x)
    if op == EXP:
        return torch.exp(x.clamp(-80.0, 80.0))
    if op == LOG:
        return torch.where(x == 0, 0.0, torch.log(x.abs()))
    if op == SQRT:
        return x.abs().sqrt()
    if op == SQUARE:
        return x * x
    if op == RECIP:
        return 1.0 / x
    return {TAN: torch.tan, ASIN: torch.asin, ACOS: torch.acos, ATAN: torch.atan, TANH: torch.tanh}[op](x)


def _dunary64(op, x, y):
    if op == SIN:
        return torch.cos(x)
    if op == COS:
        return -torch.sin(x)
    if op == EXP:
        return torch.where((x > 80) | (x < -80), 0.0, y)
    if op == LOG:
        return torch.where(x == 0, 0.0, 1.0 / x)
    if op == SQRT:
        return torch.where(x == 0, 0.0, torch.sign(x) * 0.5 / y)
    if op == SQUARE:
        return 2 * x
    if op == RECIP:
        return -y * y
    if op == TAN:
        return 1 + y * y
    if op == ASIN:
        return 1 / ((1 - x) * (1 + x)).sqrt()
    if op == ACOS:
        return -1 / ((1 - x) * (1 + x)).sqrt()
    if op == ATAN:
        return 1 / (1 + x * x)
    e = torch.exp(-2 * x.abs())
    return 4 * e / (1 + e) ** 2


def _binary64(op, a, b):
    if op == ADD:
        return a + b
    if op == SUB:
        return a - b
    if op == MUL:
        return a * b
    return torch.where(b == 0, 1.0, a / b)


def _dbinary64(op, a, b):
    one = torch.ones_like(a)
    if op == ADD:
        return one, one
    if op == SUB:
        return one, -one
    if op == MUL:
        return b, a
    z = b == 0
    return torch.where(z, 0.0, 1.0 / b), torch.where(z, 0.0, -a / (b * b))


def _range32(v):
    """A binary64 value over the binary32 range: beyond it an infinity, below
    its subnormal numbers zero (the programs' classes are those of binary32)."""
    v = torch.where(v.abs() < 2.0 ** -150, 0.0, v)
    return torch.where(v.abs() >= 2.0 ** 128, v * float("inf"), v)


class _Plan:
    """A group of programs position by position: per operator the programs
    that hold it there, and the position of each token's left operand."""

    def __init__(self, tok, consts, const_offset):
        n, T = tok.shape
        dev = tok.device
        op = torch.where(tok >= 0, tok & 0xFF, -1)
        arg = tok >> 8
        L = (tok >= 0).sum(1)
        start = torch.zeros((n, T), dtype=torch.int64, device=dev)
        left = torch.zeros((n, T), dtype=torch.int64, device=dev)
        rows = torch.arange(n, device=dev)
        for t in range(T):
            o = op[:, t]
            unary = (o >= SIN) & (o != VAR) & (o != CONST)
            prev = start[:, t - 1] if t else start[:, 0]
            left[:, t] = (prev - 1).clamp(min=0)
            start[:, t] = torch.where(o < 0, t, torch.where(unary, prev, t))
            binary = (o >= 0) & (o < 4)
            start[:, t] = torch.where(binary, start[rows, left[:, t]], start[:, t])
        self.n, self.T, self.root, self.left, self.arg = n, T, L - 1, left, arg
        self.value = torch.zeros((n, T), dtype=torch.float64, device=dev)
        slot = (const_offset[:, None] + arg).clamp(0, max(consts.numel() - 1, 0))
        if consts.numel():
            self.value = torch.where(op == CONST, consts.double()[slot], 0.0)
        self.slot = torch.where(op == CONST, slot, -1)
        self.steps = []
        for t in range(T):
            at = [(o, torch.nonzero(op[:, t] == o).flatten()) for o in range(18)]
            self.steps.append([(o, i) for o, i in at if i.numel()])

    def forward(self, V, Xt):
        """V [n, T, m]: every token's value on the cases of Xt [D, m]."""
        for t, step in enumerate(self.steps):
            for o, i in step:
                if o == VAR:
                    V[i, t] = Xt[self.arg[i, t]]
                elif o == CONST:
                    V[i, t] = self.value[i, t][:, None].expand(-1, V.shape[2])
                elif o < 4:
                    V[i, t] = _range32(_binary64(o, V[i, self.left[i, t]], V[i, t - 1]))
                else:
                    V[i, t] = _range32(_unary64(o, V[i, t - 1]))
        return V[torch.arange(self.n, device=V.device), self.root]

    def reverse(self, V, seed, grad):
        """Adds the constants' gradients of seed [n, m] = dF/dyhat to grad."""
        G = torch.zeros_like(V)
        G[torch.arange(self.n, device=V.device), self.root] = seed
        for t in range(self.T - 1, -1, -1):
            for o, i in self.steps[t]:
                if o == VAR:
                    continue
                g = G[i, t]
                if o == CONST:
                    grad[self.slot[i, t]] += g.sum(1)
                elif o < 4:
                    lft = self.left[i, t]
                    da, db = _dbinary64(o, V[i, lft], V[i, t - 1])
                    G[i, lft] = g * da
                    G[i, t - 1] = g * db
                else:
                    G[i, t - 1] = g * _dunary64(o, V[i, t - 1], V[i, t])


def _groups(tok, M, arrays):
    """Program ranges and case blocks that keep a group's values within
    memory: programs in order, a whole case set per program where it fits."""
    budget = (12 << 30) // 8 // arrays
    T = tok.shape[1]
    m = min(M, max(1, budget // T))
    n = max(1, min(tok.shape[0], budget // (T * m)))
    return n, m


def _outputs64(tok, progs, X, visit, arrays=1):
    """visit(plan, programs, first case, outputs, V) per group and block."""
    N, M = tok.shape[0], X.shape[0]
    Xt = X.double().t().contiguous()
    n, m = _groups(tok, M, arrays)
    for p0 in range(0, N, n):
        sel = slice(p0, min(N, p0 + n))
        plan = _Plan(tok[sel], progs.consts, progs.const_offset[sel])
        for c0 in range(0, M, m):
            x = Xt[:, c0:c0 + m].contiguous()
            V = torch.empty((plan.n, plan.T, x.shape[1]), dtype=torch.float64, device=DEVICE)
            visit(plan, sel, c0, plan.forward(V, x), V)


def _fitness64(kind, tok, progs, X, y):
    N, M = tok.shape[0], X.shape[0]
    y64 = y.double()
    S = MAX_SCORE
    ok_y = torch.isfinite(y64)
    # one pass of sums per block; the correlation sums about the output at the
    # first case
    sums = torch.zeros((N, 8), dtype=torch.float64, device=DEVICE)
    ref = torch.zeros(N, dtype=torch.float64, device=DEVICE)
    w_all = torch.where(ok_y, y64, 0.0) - y64[ok_y].mean()

    def visit(plan, sel, c0, yh, V):
        t = y64[c0:c0 + yh.shape[1]]
        ok_t = ok_y[c0:c0 + yh.shape[1]]
        if kind == "mse":
            sums[sel, 0] += (yh - t).square().sum(1)
            return
        ok = torch.isfinite(yh)
        if kind == "point":
            a, b = yh.abs(), t.abs()
            hi, lo = torch.maximum(a, b), torch.minimum(a, b)
            q = S * (lo / torch.where(hi == 0, 1.0, hi))
            q = torch.where(yh * t.sign() < 0, q - S / 11.0, q).round()
            q = torch.where(hi == 0, S, q)
            q = torch.where(ok & ok_t, q, torch.where(ok == ok_t, S, -S))
            sums[sel, 0] += q.sum(1)
            return
        if c0 == 0:
            ref[sel] = torch.where(ok[:, 0], yh[:, 0], 0.0)
        w = w_all[c0:c0 + yh.shape[1]]
        both = ok & ok_t if kind == "r4" else torch.ones_like(ok)
        u = torch.where(both, yh - ref[sel][:, None], 0.0)
        wv = torch.where(both, w, 0.0)
        cols = ((ok != ok_t).double(), (~ok & ~ok_t).double(), u, u * u, u * wv, wv, wv * wv, both.double())
        for j, c in enumerate(cols):
            sums[sel, j] += c.sum(1)

    _outputs64(tok, progs, X, visit)
    if kind == "mse":
        return sums[:, 0] / M, None
    if kind == "point":
        return sums[:, 0], None
    c1, c2, su, suu, suw, sw, sww, n = sums.unbind(1)
    sxx, syy, sxy = suu - su * su / n, sww - sw * sw / n, suw - su * sw / n
    good = (sxx > 0) & (syy > 0) & (n >= 2)
    r = torch.where(good, sxy / (sxx * syy).sqrt(), 0.0)
    if kind == "r4":
        return S * r ** 4 * n - S * (c1 - c2), None
    bad = ~torch.isfinite(su + suu + suw)
    fit = torch.where(bad, float("nan"), torch.where(sxx > 0, (1 - r * r).clamp(0, 1), 1.0))
    alpha = torch.where(sxx > 0, -2 * r / (sxx * syy).sqrt(), 0.0)
    beta = torch.where(sxx > 0, 2 * r * r / sxx, 0.0)
    nan = torch.where(bad, float("nan"), 0.0)
    return fit, (alpha + nan, beta + nan, ref + su / n)


def _gradient64(kind, tok, progs, X, y):
    M = X.shape[0]
    y64 = y.double()
    fit, coef = _fitness64(kind, tok, progs, X, y)
    grad = torch.zeros(progs.consts.numel(), dtype=torch.float64, device=DEVICE)

    def visit(plan, sel, c0, yh, V):
        t = y64[c0:c0 + yh.shape[1]]
        if kind == "mse":
            seed = 2 * (yh - t) / M
        else:
            alpha, beta, mu = (c[sel][:, None] for c in coef)
            seed = alpha * (t - y64.mean()) + beta * (yh - mu)
        plan.reverse(V, seed, grad)

    _outputs64(tok, progs, X, visit, arrays=2)
    return fit, grad


def exact(case, seed):
    call = case["call"]
    if call in ("generation", "microcosm"):
        return None  # integers, and constants that are copied or drawn
    if call == "batched" and case["kind"] == "mse":
        return None  # a few hundred programs' errors are ruled by the one that rounding moves most
    inp = _inputs(case, seed)
    if call == "batched":
        return [_fitness64(case["kind"], *q)[0] for q in inp]
    if call == "grad":
        return _gradient64(case["kind"], *inp)
    if call == "predict":
        tok, progs, X, _ = inp
        out = torch.empty((tok.shape[0], X.shape[0]), dtype=torch.float64, device=DEVICE)

        def visit(plan, sel, c0, yh, V):
            out[sel, c0:c0 + yh.shape[1]] = yh

        _outputs64(tok, progs, X, visit)
        return out
    return _fitness64(case["kind"], *inp)[0]
