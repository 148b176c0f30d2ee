"""Performance cases: the calls a user of the library makes, over the ranges they make them in.

A case is a dict of plain values.  `listed()` gives the named cases, `draw(rng)` one more of the
same ranges, `prepare(case, seed)` the inputs of a call (the options or the basket; Heston
parameters and the Philox seed follow from the seed), `run(state)` one call and its results,
`work(case)` the bytes and FP32 operations the path cannot do without, and `exact(case, seed)`
the same results in 64-bit torch arithmetic.

Results come back as float32: the paths are simulated in FP32 (the Broadie-Kaya scheme's step
runs in FP64 on an FP32 state).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2402_12111_amd import simr, workloads

SCHEMES = {"qe": simr.SCHEME_QE, "fte": simr.SCHEME_FTE, "qe_m": simr.SCHEME_QE_M, "tg": simr.SCHEME_TG,
           "bk": simr.SCHEME_BK}
PAYOFFS = {"euro_call": simr.EURO_CALL, "euro_put": simr.EURO_PUT, "amer_put": simr.AMER_PUT,
           "amer_call": simr.AMER_CALL}
MATURITIES = (0.25, 0.5, 1.0, 2.0)


def listed():
    return [
        # one quote on demand: the smallest call, where latency and launches count
        dict(name="price_small", kind="price", scheme="qe", payoff="euro_call", K=100.0, T=1.0, steps=64, paths=8192),
        # the accuracy reference: Broadie-Kaya exact simulation in few large steps
        dict(name="price_exact_scheme", kind="price", scheme="bk", payoff="euro_call", K=100.0, T=1.0, steps=1,
             paths=65536),
        # batched pricing of a large European book, uneven maturities and path counts
        dict(name="batch_calls", kind="batch", scheme="qe", n=1024, low=16384, high=262144, american=0.0),
        # an ordinary book: European and American calls and puts, ragged sizes
        dict(name="batch_mixed", kind="batch", scheme="qe", n=24, low=8192, high=65536, american=0.5),
        # the paper's Table 1 sizes: A American puts x N steps x 25,000 paths
        dict(name="table1_small", kind="table1", scheme="qe", n=10, steps=126, paths=25000),
        dict(name="table1_large", kind="table1", scheme="qe", n=30, steps=504, paths=25000),
        # price and adjoint Greeks of one European option (the forward and the reverse pass)
        dict(name="greeks_euro", kind="greeks", scheme="qe", payoff="euro_put", K=100.0, T=1.0, steps=252,
             paths=262144),
        # the same with d/dT and gamma under another scheme, an odd size
        dict(name="greeks_ext_odd", kind="greeks_ext", scheme="qe_m", payoff="euro_call", K=105.0, T=0.5, steps=126,
             paths=50021),
        # price and adjoint Greeks of one American option
        dict(name="greeks_american", kind="greeks", scheme="qe", payoff="amer_put", K=110.0, T=1.0, steps=252,
             paths=131072),
        # the large risk run: price and 7 Greeks of every American put of a book of underlyings
        dict(name="risk_run", kind="greeks_batch", scheme="qe", n=64, steps=252, paths=1048576),
        # a correlated basket with its deltas and cross-gammas
        dict(name="basket_greeks", kind="basket_greeks", scheme="qe", payoff="euro_call", assets=8, moneyness=1.0,
             steps=252, paths=262144),
        # an American basket of Table 1's medium size (20 assets)
        dict(name="basket_american", kind="basket_price", scheme="qe", payoff="amer_put", assets=20, moneyness=1.1,
             steps=252, paths=25000),
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(("price", "price", "exact_scheme", "batch", "batch", "table1", "greeks", "greeks", "greeks_ext",
                       "greeks_batch", "basket_greeks", "basket_price", "basket_risk"))
    if kind == "exact_scheme":
        return dict(kind="price", scheme="bk", payoff=rng.choice(("euro_call", "euro_put")),
                    K=round(rng.uniform(80.0, 120.0), 1), T=rng.choice((0.5, 1.0, 2.0)), steps=rng.randint(1, 3),
                    paths=_log_int(rng, 8192, 65536))
    T = rng.choice(MATURITIES)
    steps = int(252 * T)
    if kind == "price":
        return dict(kind=kind, scheme=rng.choice(("qe", "qe", "fte", "qe_m", "tg")),
                    payoff=rng.choice(("euro_call", "euro_put", "amer_put")), K=round(rng.uniform(85.0, 115.0), 1), T=T,
                    steps=rng.choice((steps, 64)), paths=_log_int(rng, 8192, 1 << 20))
    if kind == "batch":
        return dict(kind=kind, scheme="qe", n=_log_int(rng, 8, 128), low=8192, high=rng.choice((65536, 262144)),
                    american=rng.choice((0.0, 0.5)))
    if kind == "table1":
        return dict(kind=kind, scheme="qe", n=rng.randint(5, 30), steps=rng.choice((126, 252, 504)),
                    paths=_log_int(rng, 10000, 60000))
    if kind in ("greeks", "greeks_ext"):
        return dict(kind=kind, scheme=rng.choice(("qe", "qe", "fte", "qe_m", "tg")),
                    payoff=rng.choice(("euro_call", "euro_put", "amer_put")), K=round(rng.uniform(90.0, 115.0), 1), T=T,
                    steps=steps, paths=_log_int(rng, 16384, 1 << 19))
    if kind == "greeks_batch":
        return dict(kind=kind, scheme="qe", n=rng.randint(3, 24), steps=rng.choice((126, 252)),
                    paths=_log_int(rng, 25000, 1 << 20))
    if kind == "basket_risk":
        return dict(kind=kind, scheme=rng.choice(("qe", "fte")), payoff=rng.choice(("euro_call", "euro_put")),
                    assets=rng.randint(2, 8), moneyness=1.0, steps=rng.choice((63, 126, 252)),
                    paths=_log_int(rng, 16384, 131072))
    if kind == "basket_greeks":
        return dict(kind=kind, scheme=rng.choice(("qe", "qe", "fte", "qe_m")), payoff="euro_call",
                    assets=rng.randint(2, 16), moneyness=round(rng.uniform(0.9, 1.1), 2),
                    steps=rng.choice((63, 126, 252)), paths=_log_int(rng, 10000, 262144))
    payoff, moneyness = rng.choice((("euro_call", 1.0), ("euro_put", 1.0), ("amer_put", 1.1)))
    return dict(kind=kind, scheme="qe", payoff=payoff, assets=rng.randint(2, 32), moneyness=moneyness,
                steps=rng.choice((63, 126, 252)), paths=_log_int(rng, 10000, 131072))


# ------------------------------------------------------------------------------------------------
# Inputs: Heston parameters from the ranges of workloads.c3_batch, one Philox seed per state.
# ------------------------------------------------------------------------------------------------
def _heston(rng, n):
    return dict(kappa=rng.uniform(0.5, 3.0, n), theta=rng.uniform(0.02, 0.09, n), xi=rng.uniform(0.1, 0.8, n),
                rho=rng.uniform(-0.9, 0.0, n), v0=rng.uniform(0.01, 0.09, n))


def _options(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind in ("price", "greeks", "greeks_ext"):
        n = 1
        K, T, P, N = [case["K"]], [case["T"]], [case["paths"]], [case["steps"]]
        payoff = [PAYOFFS[case["payoff"]]]
    elif kind == "batch":
        # the book's structure (strikes, maturities, sizes, kinds) belongs to the case, the model
        # parameters and the draws to the seed
        book = np.random.default_rng(case["n"])
        n = case["n"]
        K = book.uniform(70.0, 130.0, n)
        T = book.choice(np.array(MATURITIES), n)
        P = np.rint(np.exp(book.uniform(math.log(case["low"]), math.log(case["high"]), n))).astype(np.int64)
        N = [int(round(252 * t)) for t in T]
        amer = book.uniform(0.0, 1.0, n) < case["american"]
        call = np.ones(n, bool) if case["american"] == 0.0 else book.uniform(0.0, 1.0, n) < 0.5
        payoff = [PAYOFFS["amer_put"] if a else PAYOFFS["euro_call"] if c else PAYOFFS["euro_put"]
                  for a, c in zip(amer, call)]
    else:  # table1, greeks_batch: American puts of one size, one underlying each
        n = case["n"]
        K, T, P, N = [110.0] * n, [case["steps"] / 252.0] * n, [case["paths"]] * n, [case["steps"]] * n
        payoff = [PAYOFFS["amer_put"]] * n
    h = _heston(rng, n)
    return [simr.Option(S0=100.0, K=float(K[i]), T=float(T[i]), r=0.02, kappa=float(h["kappa"][i]),
                        theta=float(h["theta"][i]), xi=float(h["xi"][i]), rho=float(h["rho"][i]),
                        v0=float(h["v0"][i]), payoff=int(payoff[i]), steps=int(N[i]), paths=int(P[i]),
                        seed=int(seed) & 0xFFFFFFFFFFFF, stream=i) for i in range(n)]


def _basket(case, seed):
    # workloads.basket draws its parameters and takes its Philox seed from `seed`
    return simr.Basket.from_dict(workloads.basket(case["assets"], seed=int(seed), moneyness=case["moneyness"],
                                                  payoff=PAYOFFS[case["payoff"]], steps=case["steps"],
                                                  T=case["steps"] / 252.0, paths=case["paths"]))


def prepare(case, seed):
    kind = case["kind"]
    what = _basket(case, seed) if kind.startswith("basket") else _options(case, seed)
    return dict(kind=kind, scheme=SCHEMES[case["scheme"]], what=what)


def _f32(x):
    return torch.tensor(x, dtype=torch.float32)


def _of_result(r):
    return dict(price=r.price, std_err=r.std_err, flags=r.lsm_flags)


def _of_results(res):
    return dict(price=_f32([r.price for r in res]), std_err=_f32([r.std_err for r in res]),
                flags=torch.tensor([r.lsm_flags for r in res]))


def run(state):
    kind, scheme, what = state["kind"], state["scheme"], state["what"]
    if kind == "price":
        return _of_result(simr.price(what[0], scheme))
    if kind in ("batch", "table1"):
        return _of_results(simr.price_batch(what, scheme))
    if kind in ("greeks", "greeks_ext"):
        r = simr.greeks(what[0], scheme) if kind == "greeks" else simr.greeks_ext(what[0], scheme)
        return dict(_of_result(r), greeks=_f32(r.grads), greeks_se=_f32(r.grad_se))
    if kind == "greeks_batch":
        res = simr.greeks_batch(what, scheme)
        return dict(_of_results(res), greeks=_f32([r.grads for r in res]), greeks_se=_f32([r.grad_se for r in res]))
    if kind == "basket_price":
        return _of_result(simr.basket_price(what, scheme))
    if kind == "basket_greeks":
        r = simr.basket_greeks(what, scheme)
        return dict(_of_result(r), delta=_f32(r.delta), delta_se=_f32(r.delta_se), gamma=_f32(r.gamma),
                    gamma_se=_f32(r.gamma_se))
    r = simr.basket_risk(what, scheme)
    return dict(_of_result(r), vega_v0=_f32(r.vega_v0), vega_v0_se=_f32(r.vega_v0_se), vega_theta=_f32(r.vega_theta),
                vega_theta_se=_f32(r.vega_theta_se), dcorr=_f32(r.dcorr), dcorr_se=_f32(r.dcorr_se))


# FP32 operations of the method as written, a fused multiply-add counted twice and a transcendental
# once: a forward step (uniforms, Box-Muller, QE variance and log-price) 46, its adjoint step 121
# with the recomputation, a regression date (basis, right-hand sides, Gram sums, exercise) 60 on 6
# functions and 150 on 10, a Broadie-Kaya step 1e6.  Bytes: inputs and results, and for American
# options the path states, written once and read once by the backward induction (8 B each way).
def work(case):
    kind = case["kind"]
    if kind.startswith("basket"):
        d, ps = case["assets"], case["steps"] * case["paths"]
        amer = case["payoff"].startswith("amer")
        flops = ps * (46 * d + d * (d + 1))
        if kind == "basket_greeks":
            flops += ps * (d * (d + 1) + 4 * d)
        if kind == "basket_risk":
            flops += ps * (60 * d + d * (d + 1))
        return dict(bytes=9000 + (16.0 * ps if amer else 0), flops=float(flops + (150 * ps if amer else 0)))
    opts = _options(case, 0)
    flops = bytes_ = 0.0
    for o in opts:
        ps = o.steps * o.paths
        amer = o.payoff in (simr.AMER_PUT, simr.AMER_CALL)
        flops += ps * (1e6 if case["scheme"] == "bk" else 46 + (60 if amer else 0))
        bytes_ += 120 + (16.0 * ps if amer else 0)
        if kind.startswith("greeks"):
            flops += ps * 121
    return dict(bytes=bytes_, flops=flops)


# ------------------------------------------------------------------------------------------------
# The same results in 64 bits: plain torch, one vector element per path.
# ------------------------------------------------------------------------------------------------
MASK = 0xFFFFFFFF


def _hi(p):
    return (p >> 32) & MASK


def _philox(c0, c1, c2, c3, seed):
    k0, k1 = seed & MASK, (seed >> 32) & MASK
    for _ in range(10):
        pa, pb = 0xD2511F53 * c0, 0xCD9E8D57 * c2
        c0, c1, c2, c3 = _hi(pb) ^ c1 ^ k0, pb & MASK, _hi(pa) ^ c3 ^ k1, pa & MASK
        k0, k1 = (k0 + 0x9E3779B9) & MASK, (k1 + 0xBB67AE85) & MASK
    return c0, c1, c2


def _draws(n, path, stream, asset, seed):
    u = [((w >> 9).double() + 0.5) * 2.0 ** -23 for w in _philox(n, path, stream, asset, seed)]
    r = torch.sqrt(-2.0 * torch.log(u[0]))
    return r * torch.cos(2.0 * math.pi * u[1]), r * torch.sin(2.0 * math.pi * u[1]), u[2]


def _sqrt0(w):
    """sqrt with derivative 0 at 0."""
    pos = w > 0
    return torch.where(pos, torch.sqrt(torch.where(pos, w, 1.0)), 0.0)


class _Model:
    """Step constants of one asset in 64 bits; every parameter a tensor (per path or 0-d)."""

    def __init__(self, scheme, p, N):
        self.scheme, self.p = scheme, p
        dt = p["T"] / N
        kappa, theta, xi, rho, r = p["kappa"], p["theta"], p["xi"], p["rho"], p["r"]
        self.dt, self.E = dt, torch.exp(-kappa * dt)
        omE = -torch.expm1(-kappa * dt)
        self.A1 = xi * xi * self.E * omE / kappa
        self.A2 = theta * xi * xi * omE * omE / (2.0 * kappa)
        self.C0 = r * dt - rho * kappa * theta * dt / xi
        self.K1 = 0.5 * dt * (kappa * rho / xi - 0.5) - rho / xi
        self.K2 = 0.5 * dt * (kappa * rho / xi - 0.5) + rho / xi
        self.K3 = 0.5 * dt * (1.0 - rho * rho)

    def step(self, x, v, z1, z2, u):
        """(x', v', coefficient of z2 in the log-price increment)."""
        p = self.p
        if self.scheme == "fte":
            vp = torch.clamp(v, min=0.0)
            sv = _sqrt0(vp) * torch.sqrt(self.dt)
            srho = torch.sqrt(1.0 - p["rho"] ** 2)
            xn = x + p["r"] * self.dt - 0.5 * vp * self.dt + sv * (p["rho"] * z1 + srho * z2)
            return xn, v + p["kappa"] * (p["theta"] - vp) * self.dt + p["xi"] * sv * z1, sv * srho
        m = p["theta"] + (v - p["theta"]) * self.E
        s2 = v * self.A1 + self.A2
        psi = s2 / (m * m)
        quad = psi <= 1.5
        t = 2.0 / torch.where(quad, psi, 1.0)
        b2 = (t - 1.0) + torch.sqrt(t * (t - 1.0))
        a = m / (1.0 + b2)
        pe = torch.where(quad, 2.0, psi)
        q = (pe - 1.0) / (pe + 1.0)
        L = torch.log((1.0 - q) / (1.0 - u))
        V = torch.where(quad, a * (torch.sqrt(b2) + z1) ** 2, torch.where(u <= q, 0.0, L * m / (1.0 - q)))
        c0 = self.C0
        if self.scheme == "qe_m":
            A = self.K2 + 0.5 * self.K3
            dd = 1.0 - 2.0 * A * a
            ds = torch.where(quad & (dd > 0), dd, 1.0)
            beta = (1.0 - q) / m
            ok = torch.where(quad, dd > 0, A < beta)
            gap = torch.where(~quad & ok, beta - A, 1.0)
            g = torch.where(quad, A * b2 * a / ds - 0.5 * torch.log(ds),
                            torch.log(torch.where(ok & ~quad, q + beta * (1.0 - q) / gap, 1.0)))
            c0 = torch.where(ok, p["r"] * self.dt - (self.K1 + 0.5 * self.K3) * v - g, c0)
        s = _sqrt0(self.K3 * (v + V))
        return x + c0 + self.K1 * v + self.K2 * V + s * z2, V, s


def _payoff(kind, S, K):
    return torch.clamp(S - K if kind in (simr.EURO_CALL, simr.AMER_CALL) else K - S, min=0.0)


def _mean_se(X):
    n = X.shape[0]
    m = X.mean(0)
    return m, torch.sqrt(torch.clamp((X * X).mean(0) - m * m, min=0.0) / (n - 1))


def _lsm(S, v, K, theta, r, dt, payoff, nb):
    """(cash flows valued at t_0, exercise dates, flags) of the in-sample regression rule; S, v: [N, P]."""
    N, P = S.shape
    tau = torch.full((P,), N, device=S.device)
    w = _payoff(payoff, S[N - 1], K) * math.exp(-r * N * dt)
    flags = 0
    for n in range(N - 1, 0, -1):
        h = _payoff(payoff, S[n - 1], K)
        itm = h > 0
        a, c = S[n - 1] / K - 1.0, torch.clamp(v[n - 1], min=0.0) / theta - 1.0
        phi = [torch.ones_like(a), a, a * a, c, a * c, c * c]
        if nb == 10:
            phi += [a ** 3, a * a * c, a * c * c, c ** 3]
        phi = torch.stack(phi, 1)
        pm = phi * itm[:, None]
        if int(itm.sum()) < nb:
            flags |= 1
            continue
        y = pm.T @ (w * math.exp(r * n * dt))
        G = (pm.T @ phi).cpu()
        beta = torch.linalg.solve(G, y.cpu()).to(S.device)
        ex = itm & (h > phi @ beta)
        w = torch.where(ex, h * math.exp(-r * n * dt), w)
        tau = torch.where(ex, n, tau)
    return w, tau, flags


CHUNK = 65536  # paths differentiated together: about 10 GB of 64-bit intermediates at 252 steps


def _forward(scheme, o, keep):
    """(x_N, [x_n], [v_n]) of one option."""
    dev = torch.device("cuda")
    p = {k: torch.tensor(getattr(o, k), dtype=torch.float64, device=dev)
         for k in ("T", "r", "kappa", "theta", "xi", "rho")}
    model = _Model(scheme, p, o.steps)
    path = torch.arange(o.paths, device=dev)
    x, v = torch.zeros(o.paths, dtype=torch.float64, device=dev), torch.full((o.paths,), o.v0, dtype=torch.float64, device=dev)
    xs, vs = [], []
    for n in range(o.steps):
        x, v, _ = model.step(x, v, *_draws(n, path, o.stream, 0, o.seed))
        if keep:
            xs.append(x)
            vs.append(v)
    return x, xs, vs


GREEKS = ("S0", "v0", "theta", "r", "kappa", "xi", "rho", "T")


def _path_greeks(scheme, o, tau, ext):
    """Per-path derivatives of e^{-r tau dt} h(S_tau) in the model parameters (and T, and gamma)."""
    dev = torch.device("cuda")
    out = []
    for lo in range(0, o.paths, CHUNK):
        path = torch.arange(lo, min(lo + CHUNK, o.paths), device=dev)
        p = {k: torch.full(path.shape, getattr(o, k), dtype=torch.float64, device=dev, requires_grad=True)
             for k in GREEKS}
        model = _Model(scheme, p, o.steps)
        stop = torch.full(path.shape, o.steps, device=dev) if tau is None else tau[lo:lo + CHUNK]
        x, v = torch.zeros(path.shape, dtype=torch.float64, device=dev), p["v0"]
        sz = ss = 0.0
        for n in range(int(stop.max())):
            z1, z2, u = _draws(n, path, o.stream, 0, o.seed)
            xn, v, s = model.step(x, v, z1, z2, u)
            x = torch.where(n < stop, xn, x)
            with torch.no_grad():
                sz, ss = sz + s * z2, ss + s * s
        S = p["S0"] * torch.exp(x)
        X = torch.exp(-p["r"] * stop * (p["T"] / o.steps)) * _payoff(o.payoff, S, o.K)
        g = list(torch.autograd.grad(X.sum(), [p[k] for k in GREEKS], allow_unused=True))
        if ext:
            gamma = g[0] * o.S0 * (sz / ss - 1.0) / o.S0 ** 2 if tau is None else torch.full_like(x, math.nan)
            g.append(gamma.detach())
        else:
            g = g[:7]
        out.append(torch.stack([t.detach() for t in g], 1))
    return torch.cat(out)


def _exact_option(case, o, greeks):
    """(price, std_err, flags, greeks, greeks_se) of one option."""
    scheme = case["scheme"]
    amer = o.payoff in (simr.AMER_PUT, simr.AMER_CALL)
    x, xs, vs = _forward(scheme, o, amer)
    tau, flags = None, 0
    if amer:
        S = o.S0 * torch.exp(torch.stack(xs))
        X, tau, flags = _lsm(S, torch.stack(vs), o.K, o.theta, o.r, o.T / o.steps, o.payoff, 6)
    else:
        X = math.exp(-o.r * o.T) * _payoff(o.payoff, o.S0 * torch.exp(x), o.K)
    price, se = (float(t) for t in _mean_se(X))
    h0 = max(0.0, (o.S0 - o.K) if o.payoff == simr.AMER_CALL else (o.K - o.S0))
    at_t0 = amer and h0 > price
    if at_t0:
        price, se, flags = h0, 0.0, flags | simr.LSM_EXERCISE_T0
    del xs, vs
    if not greeks:
        return price, se, flags, None, None
    ext = case["kind"] == "greeks_ext"
    ng = 9 if ext else 7
    if at_t0:
        return price, se, flags, [-1.0] + [0.0] * (ng - 1), [0.0] * ng
    g, gs = _mean_se(_path_greeks(scheme, o, tau, ext))
    return price, se, flags, g.tolist(), gs.tolist()


def _exact_basket(case, b):
    dev = torch.device("cuda")
    f64 = dict(dtype=torch.float64, device=dev)
    kind, scheme, d, N = case["kind"], case["scheme"], b.assets, b.steps
    amer = b.payoff in (simr.AMER_PUT, simr.AMER_CALL)
    risk, greeks = kind == "basket_risk", kind == "basket_greeks"
    C = torch.tensor(b.corr, dtype=torch.float64)
    L = torch.linalg.cholesky(C).to(dev)
    Linv = torch.linalg.inv(L)
    w = torch.tensor(b.w, **f64)
    S0 = torch.tensor(b.S0, **f64)
    B0 = float((w * S0).sum())
    cols = {k: [] for k in ("X", "D", "G", "v0", "theta", "L")}
    Bs, vbars = [], []
    chunk = b.paths if not risk else 8192
    for lo in range(0, b.paths, chunk):
        path = torch.arange(lo, min(lo + chunk, b.paths), device=dev)
        P = path.shape[0]
        models, x, v, leaf = [], [], [], []
        Lp = L.expand(P, d, d).clone().requires_grad_(True) if risk else None
        for i in range(d):
            p = {k: torch.tensor(getattr(b, k)[i], **f64) for k in ("kappa", "theta", "xi", "rho")}
            p["T"], p["r"] = torch.tensor(b.T, **f64), torch.tensor(b.r, **f64)
            v0 = torch.full((P,), b.v0[i], **f64)
            if risk:
                p["theta"] = torch.full((P,), b.theta[i], **f64).requires_grad_(True)
                v0.requires_grad_(True)
                leaf.append((v0, p["theta"]))
            models.append(_Model(scheme, p, N))
            x.append(torch.zeros(P, **f64))
            v.append(v0)
        num = [0.0] * d
        den = [0.0] * d
        for n in range(N):
            z1, z2, u = zip(*[_draws(n, path, b.stream, i, b.seed) for i in range(d)])
            z2 = torch.stack(z2, 1)
            zc = (Lp * z2[:, None, :]).sum(2) if risk else z2 @ L.T
            ut = z2 @ Linv if greeks else None  # (L^{-T} z2)_j
            for i in range(d):
                x[i], v[i], s = models[i].step(x[i], v[i], z1[i], zc[:, i], u[i])
                if greeks:
                    num[i], den[i] = num[i] + s * ut[:, i], den[i] + s * s
            if amer:
                Si = [w[i] * S0[i] * torch.exp(x[i]) for i in range(d)]
                Bs.append(sum(Si))
                vbars.append(sum(Si[i] * torch.clamp(v[i], min=0.0) for i in range(d)) / Bs[-1])
        e = torch.exp(torch.stack(x, 1))
        B = (w * S0 * e).sum(1)
        X = math.exp(-b.r * b.T) * _payoff(b.payoff, B, b.K)
        cols["X"].append(X.detach())
        if greeks:
            slope = torch.where(X > 0, math.exp(-b.r * b.T) * (1.0 if b.payoff == simr.EURO_CALL else -1.0), 0.0)
            D = slope[:, None] * w * e
            W = torch.stack(num, 1) / torch.stack(den, 1)
            G = 0.5 * (D[:, :, None] * (W / S0)[:, None, :] + (W / S0)[:, :, None] * D[:, None, :])
            cols["D"].append(D)
            cols["G"].append(G - torch.diag_embed(D / S0))
        if risk:
            g = torch.autograd.grad(X.sum(), [q for pair in leaf for q in pair] + [Lp])
            cols["v0"].append(torch.stack(g[0:2 * d:2], 1))
            cols["theta"].append(torch.stack(g[1:2 * d:2], 1))
            cols["L"].append(g[-1])
    X, flags = torch.cat(cols["X"]), 0
    if amer:
        thbar = sum(b.w[i] * b.S0[i] * b.theta[i] for i in range(d)) / B0
        X, _, flags = _lsm(torch.stack(Bs), torch.stack(vbars), b.K, thbar, b.r, b.T / N, b.payoff, 10)
    price, se = (float(t) for t in _mean_se(X))
    if amer and b.K - B0 > price:
        price, se, flags = b.K - B0, 0.0, flags | simr.LSM_EXERCISE_T0
    out = dict(price=price, std_err=se, flags=flags)
    if greeks:
        for name, key in (("delta", "D"), ("gamma", "G")):
            out[name], out[name + "_se"] = _mean_se(torch.cat(cols[key]))
    if risk:
        for name in ("v0", "theta"):
            out["vega_" + name], out["vega_" + name + "_se"] = _mean_se(torch.cat(cols[name]))
        dL = torch.cat(cols["L"])
        out["dcorr"], out["dcorr_se"] = torch.zeros(d, d, **f64), torch.zeros(d, d, **f64)
        for i in range(d):
            for j in range(i):
                move = torch.zeros(d, d, dtype=torch.float64)
                move[i, j] = move[j, i] = 1.0
                _, t = torch.autograd.functional.jvp(torch.linalg.cholesky, C, move)
                m, s = _mean_se((dL * t.to(dev)).sum((1, 2)))
                out["dcorr"][i, j] = out["dcorr"][j, i] = m
                out["dcorr_se"][i, j] = out["dcorr_se"][j, i] = s
    return out


def exact(case, seed):
    kind = case["kind"]
    if case["scheme"] in ("tg", "bk"):  # roots of special functions at every step
        return None
    if kind.startswith("basket"):
        cost = case["steps"] * case["assets"] * (1 + case["paths"] / 2e5) * (max(1.0, case["paths"] / 3e4) if kind == "basket_risk" else 1.0)
        return None if cost > 8000 else _exact_basket(case, _basket(case, seed))
    opts = _options(case, seed)
    greeks = kind.startswith("greeks")
    # seconds: about 2 ms a step, more for many paths, and the reverse passes
    cost = sum(o.steps * (2e-3 + o.paths * 6e-9 + (1 + o.paths // CHUNK) * 6e-3 * greeks) for o in opts)
    if cost > 18.0:
        return None
    res = [_exact_option(case, o, greeks) for o in opts]
    if kind in ("price", "greeks", "greeks_ext"):
        out = dict(price=res[0][0], std_err=res[0][1], flags=res[0][2])
        if greeks:
            out.update(greeks=torch.tensor(res[0][3], dtype=torch.float64),
                       greeks_se=torch.tensor(res[0][4], dtype=torch.float64))
        return out
    f64 = torch.float64
    out = dict(price=torch.tensor([r[0] for r in res], dtype=f64), std_err=torch.tensor([r[1] for r in res], dtype=f64),
               flags=torch.tensor([r[2] for r in res]))
    if greeks:
        out.update(greeks=torch.tensor([r[3] for r in res], dtype=f64),
                   greeks_se=torch.tensor([r[4] for r in res], dtype=f64))
    return out
