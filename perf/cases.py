"""The work that users of this framework have it do, as timed cases.

Every case is one call (or one forward and backward pass) of a public entry
point at sizes of the repository's own workloads, tests and benchmark, or at
ragged ones between them. A case's "kind" names the path, and draw() gives
further sizes of the same kinds, none of them larger than the listed one of
its kind. Market parameters and the Philox key come from the seed.

exact() is the same estimate in plain torch and numpy at 64 bits: the
documented random-number layout (Philox4x32-10, Box-Muller, Sobol' points)
and the estimators' formulas, without the package.
"""
import math
import random

import numpy as np
import torch

import paper_1906_02818_amd as mc

PAYOFFS = {"euro": mc.MC_EURO_CALL, "asian": mc.MC_ASIAN_ARITH_CALL,
           "uo": mc.MC_UO_BARRIER_CALL, "bridge": mc.MC_UO_BRIDGE_CALL}
PRECS = {"fp64": mc.MC_FP64, "fp32": mc.MC_FP32, "bf16": mc.MC_BF16_GEMM, "fp16": mc.MC_FP16_GEMM,
         "bf16x2": mc.MC_BF16X2_GEMM}
METHODS = {"pathwise": mc.MC_GREEKS_PATHWISE, "tangent": mc.MC_GREEKS_TANGENT,
           "fd": mc.MC_GREEKS_FD_CRN}


def listed():
    return [
        # The smallest call: a quote of a monthly-fixing Asian with its
        # control variate on a few thousand paths, where latency counts.
        dict(name="quote_asian_cv", kind="gbm", payoff="asian", prec="fp32", greeks="", cv=True,
             n_paths=8192, n_steps=12),
        # A European call with its greeks in double precision, the
        # benchmark's 2^18 x 64.
        dict(name="euro_fp64_greeks", kind="gbm", payoff="euro", prec="fp64", greeks="pathwise",
             cv=False, n_paths=1 << 18, n_steps=64),
        # Asian with control variate, geometric Asian and barrier on one set
        # of paths: the benchmark's default workload, the largest case.
        dict(name="asian_barrier_multi", kind="multi", n_paths=1 << 24, n_steps=252),
        # Barrier greeks exist as finite differences only (double-precision
        # bumped pairs); a ragged path count and weekly monitoring.
        dict(name="barrier_fd_greeks", kind="gbm", payoff="uo", prec="fp32", greeks="fd", cv=False,
             n_paths=300007, n_steps=52),
        # Heston Asian with delta and vega at the benchmark's 2^22 x 256.
        dict(name="heston_greeks", kind="heston", payoff="asian", prec="fp32", greeks="pathwise",
             n_paths=1 << 22, n_steps=256),
        # The Heston price as a differentiable function in a torch program:
        # forward and backward, ragged sizes.
        dict(name="heston_autograd", kind="autograd", payoff="euro", n_paths=500009, n_steps=100),
        # Pricing with a trained hedge network, rebalanced every 16 steps.
        dict(name="learned_cv_price", kind="cv_price", prec="bf16", hedge_every=16, n_paths=1 << 21,
             n_steps=256),
        # Training that network: the benchmark's minibatch, 32 of its Adam
        # steps on a part of its training set.
        dict(name="learned_cv_train", kind="cv_train", prec="bf16", hedge_every=16,
             n_train=1 << 18, batch=1 << 15, adam_steps=32, n_steps=256),
        # Basket of 256 assets, 100 steps, with its delta: the benchmark's
        # market and precision on a quarter of its paths.
        dict(name="basket_bf16", kind="basket", prec="bf16", d=256, n_paths=1 << 18, n_steps=100),
        # Value at risk of a call portfolio in single precision, a middle-
        # sized market and a ragged number of scenarios.
        dict(name="risk_fp32", kind="risk", prec="fp32", d=112, n_paths=100003, n_steps=50),
        # Randomised quasi-Monte Carlo on 16 assets, the benchmark's 16 x 2^16.
        dict(name="qmc_basket", kind="qmc", prec="fp32", d=16, n_paths=1 << 16, n_steps=1,
             replicates=16),
        # Bermudan max-call by Longstaff-Schwartz with its out-of-sample
        # estimate, the benchmark's contract on a quarter of its paths.
        dict(name="lsm_max_call", kind="lsm", payoff="max_call", d=2, degree=2, n_dates=9,
             steps_per_date=1, n_paths=1 << 22, n_oos=1 << 22),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["gbm", "gbm", "multi", "heston", "heston", "autograd", "cv_price",
                       "cv_train", "basket", "basket", "risk", "qmc", "lsm"])
    if kind == "gbm":
        form = rng.choice(["quote", "fp64", "fd"])
        if form == "quote":
            return dict(kind=kind, payoff=rng.choice(["euro", "asian", "uo", "bridge"]),
                        prec="fp32", greeks="", cv=False, n_paths=_log_int(rng, 1000, 200000),
                        n_steps=_log_int(rng, 4, 60))
        if form == "fp64":
            return dict(kind=kind, payoff=rng.choice(["euro", "asian"]), prec="fp64",
                        greeks=rng.choice(["", "pathwise"]), cv=False,
                        n_paths=_log_int(rng, 20000, 1 << 18), n_steps=rng.randint(8, 64))
        return dict(kind=kind, payoff=rng.choice(["uo", "bridge"]), prec="fp32", greeks="fd",
                    cv=False, n_paths=_log_int(rng, 20000, 300000), n_steps=rng.randint(8, 52))
    if kind == "multi":
        return dict(kind=kind, n_paths=_log_int(rng, 1 << 18, 1 << 24), n_steps=rng.randint(12, 252))
    if kind == "heston":
        return dict(kind=kind, payoff=rng.choice(["asian", "euro"]), prec="fp32",
                    greeks=rng.choice(["", "pathwise", "tangent"]),
                    n_paths=_log_int(rng, 1 << 15, 1 << 22), n_steps=rng.randint(12, 256))
    if kind == "autograd":
        return dict(kind=kind, payoff=rng.choice(["asian", "euro"]),
                    n_paths=_log_int(rng, 10000, 500000), n_steps=rng.randint(12, 100))
    if kind == "cv_price":
        return dict(kind=kind, prec=rng.choice(["bf16", "fp32"]),
                    hedge_every=rng.choice([16, 20, 24, 32]),
                    n_paths=_log_int(rng, 1 << 16, 1 << 20), n_steps=rng.randint(48, 256))
    if kind == "cv_train":
        batch = 256 * rng.choice([16, 24, 32, 56, 64, 100, 128])
        return dict(kind=kind, prec=rng.choice(["bf16", "fp32"]),
                    hedge_every=rng.choice([16, 20, 24, 32]), n_train=batch * rng.randint(2, 4),
                    batch=batch, adam_steps=rng.randint(8, 24), n_steps=rng.randint(48, 256))
    if kind == "basket":
        # Reduced precision where it is used: many assets and many paths.
        prec = rng.choice(["bf16", "fp32", "fp16", "bf16x2"])
        return dict(kind=kind, prec=prec, d=16 * rng.randint(1, 12),
                    n_paths=_log_int(rng, 1 << 16, 1 << 18), n_steps=rng.randint(1, 30))
    if kind == "risk":
        return dict(kind=kind, prec="fp32", d=16 * rng.randint(1, 7),
                    n_paths=_log_int(rng, 5000, 100000), n_steps=rng.randint(1, 50))
    if kind == "qmc":
        return dict(kind=kind, prec=rng.choice(["fp32", "fp16"]), d=16, n_steps=1,
                    n_paths=_log_int(rng, 4096, 1 << 16), replicates=rng.randint(2, 16))
    return dict(kind="lsm", payoff=rng.choice(["max_call", "put"]), d=rng.randint(1, 2),
                degree=rng.randint(1, 2), n_dates=rng.randint(3, 9), steps_per_date=1,
                n_paths=_log_int(rng, 1 << 16, 1 << 22), n_oos=_log_int(rng, 1 << 14, 1 << 20))


# --------------------------------------------------------------- inputs ----
def _market(case, seed):
    """Market parameters around the repository's workloads, and the key."""
    r = np.random.default_rng([seed, 1906])
    u = lambda lo, hi: float(r.uniform(lo, hi))
    m = dict(key=int(r.integers(1 << 40)), S0=u(95, 105), K=u(98, 102), T=1.0, rate=u(0.01, 0.06),
             sigma=u(0.18, 0.28), B=u(125, 140))
    if case["kind"] in ("heston", "autograd", "cv_price", "cv_train"):
        m.update(v0=u(0.035, 0.05), kappa=u(1.5, 2.5), theta=u(0.035, 0.05), xi=u(0.4, 0.55),
                 rho=u(-0.8, -0.6), rate=u(0.01, 0.03))
    d = case.get("d", 1)
    if case["kind"] in ("basket", "risk", "qmc"):
        G = r.standard_normal((d, d))
        C = 0.3 + 0.7 * np.eye(d) + 0.1 * (G @ G.T) / d
        s = 1.0 / np.sqrt(np.diag(C))
        C = C * s[:, None] * s[None, :]
        C = 0.5 * (C + C.T)
        np.fill_diagonal(C, 1.0)
        m.update(S0=[m["S0"]] * d, sigma=list(0.1 + 0.3 * r.random(d)), corr=C,
                 mu=list(np.linspace(0.02, 0.10, d)))
    if case["kind"] == "lsm":
        C = np.eye(d)
        if d == 2:
            C[0, 1] = C[1, 0] = u(-0.2, 0.3)
        m.update(S0=[u(95, 105) for _ in range(d)], sigma=[u(0.18, 0.25) for _ in range(d)], corr=C,
                 K=100.0, T=3.0, rate=0.05, q=0.1 if case["payoff"] == "max_call" else 0.0)
    return m


def _hedge_weights(m, seed):
    """A hedge network as training leaves one: its last layer fitted to the
    Black-Scholes-like delta of the running average, the layers below random."""
    r = np.random.default_rng([seed, 4])
    W1 = r.uniform(-0.8, 0.8, (64, 4))
    W1[:, 1] *= 3.0
    W1[:, 3] *= 3.0
    b1 = r.uniform(-0.5, 0.5, 64)
    W2 = r.uniform(-0.3, 0.3, (64, 64))
    b2 = r.uniform(-0.3, 0.3, 64)
    n = 4096
    t = r.random(n)
    x = 0.2 * np.sqrt(t) * r.standard_normal(n)
    v = r.gamma(2.0, 0.5, n)
    a = 0.6 * x + 0.03 * r.standard_normal(n)
    phi = np.stack([t, x, v, a], 1)
    sd = 0.2 * (1.0 - t) + 0.02
    z = (t * a + (1.0 - t) * x) / sd
    target = (1.0 - t) * np.array([0.5 * math.erfc(-q / math.sqrt(2.0)) for q in z])
    h = np.tanh(np.tanh(phi @ W1.T + b1) @ W2.T + b2)
    A = np.concatenate([h, np.ones((n, 1))], 1)
    w = np.linalg.solve(A.T @ A + 1e-2 * n * np.eye(65), A.T @ target)
    return np.concatenate([W1.ravel(), b1, W2.ravel(), b2, w]).astype(np.float32)


def _glorot(seed):
    r = np.random.default_rng([seed, 3])
    g = lambda o, i: r.uniform(-math.sqrt(6.0 / (i + o)), math.sqrt(6.0 / (i + o)), (o, i)).ravel()
    return np.concatenate([g(64, 4), np.zeros(64), g(64, 64), np.zeros(64), g(1, 64),
                           np.zeros(1)]).astype(np.float32)


ADAM = dict(lr=2e-3, beta1=0.9, beta2=0.95, eps=1e-8)
PORTFOLIO = ((0.9, 0.95, 1.0, 1.05, 1.1), (1.0, 2.0, 1.5, 1.0, 0.5))   # long calls


def prepare(case, seed):
    m = _market(case, seed)
    kind, prec = case["kind"], PRECS[case.get("prec", "fp32")]
    st = dict(case=case, m=m, ctx=mc.mc_create(0), key=m["key"])
    heston = lambda: mc.Model(kind=mc.MC_HESTON, S0=m["S0"], r=m["rate"], T=m["T"], v0=m["v0"],
                              kappa=m["kappa"], theta=m["theta"], xi=m["xi"], rho=m["rho"])
    both = mc.MC_GREEK_DELTA | mc.MC_GREEK_VEGA
    if kind == "gbm":
        st["model"] = mc.Model(kind=mc.MC_GBM, S0=m["S0"], r=m["rate"], T=m["T"], sigma=m["sigma"])
        st["payoff"] = mc.Payoff(PAYOFFS[case["payoff"]], K=m["K"], B=m["B"],
                                 cv=mc.MC_CV_GEO_ASIAN if case["cv"] else mc.MC_CV_NONE)
        st["opts"] = mc.Options(prec=prec, greeks=both if case["greeks"] else 0,
                                greeks_method=METHODS[case["greeks"] or "pathwise"],
                                pilot_paths=mc.MC_PILOT_IN_SAMPLE if case["cv"] else 0)
    elif kind == "multi":
        model = mc.Model(kind=mc.MC_GBM, S0=m["S0"], r=m["rate"], T=m["T"], sigma=m["sigma"])
        fs = [mc.Payoff(mc.MC_ASIAN_ARITH_CALL, K=m["K"], cv=mc.MC_CV_GEO_ASIAN),
              mc.Payoff(mc.MC_UO_BARRIER_CALL, K=m["K"], B=m["B"]),
              mc.Payoff(mc.MC_ASIAN_GEO_CALL, K=m["K"])]
        st["call"] = mc.PreparedPriceMulti(st["ctx"], model, fs, case["n_paths"], case["n_steps"],
                                           st["key"], mc.Options(pilot_paths=mc.MC_PILOT_IN_SAMPLE))
    elif kind == "heston":
        st["model"] = heston()
        st["payoff"] = mc.Payoff(PAYOFFS[case["payoff"]], K=m["K"])
        st["opts"] = mc.Options(prec=prec, greeks=both if case["greeks"] else 0,
                                greeks_method=METHODS[case["greeks"] or "pathwise"])
    elif kind == "autograd":
        st["model"] = heston()
        st["payoff"] = mc.Payoff(PAYOFFS[case["payoff"]], K=m["K"])
    elif kind == "cv_price":
        st["model"] = heston()
        st["payoff"] = mc.Payoff(mc.MC_ASIAN_ARITH_CALL, K=m["K"], cv=mc.MC_CV_LEARNED)
        st["opts"] = mc.Options(prec=prec, cv_weights=_hedge_weights(m, seed),
                                cv_hedge_every=case["hedge_every"], cv_beta=1.0)
    elif kind == "cv_train":
        st["model"] = heston()
        st["payoff"] = mc.Payoff(mc.MC_ASIAN_ARITH_CALL, K=m["K"])
        st["weights"] = _glorot(seed)
    elif kind in ("basket", "risk", "qmc"):
        st["model"] = mc.Model(kind=mc.MC_GBM_BASKET, S0=m["S0"], r=m["rate"], T=m["T"],
                               sigma=m["sigma"], corr=m["corr"])
        st["payoff"] = mc.Payoff(mc.MC_BASKET_CALL, K=m["K"])
        st["opts"] = mc.Options(prec=prec, greeks=mc.MC_GREEK_DELTA if kind == "basket" else 0)
    else:
        d = case["d"]
        st["model"] = mc.Model(kind=mc.MC_GBM if d == 1 else mc.MC_GBM_BASKET, S0=m["S0"],
                               r=m["rate"], T=m["T"], sigma=m["sigma"],
                               corr=m["corr"] if d > 1 else None)
        pay = mc.MC_LSM_MAX_CALL if case["payoff"] == "max_call" else mc.MC_LSM_BASKET_PUT
        st["spec"] = mc.LsmSpec(payoff=pay, K=m["K"], dividend=m["q"], n_dates=case["n_dates"],
                                steps_per_date=case["steps_per_date"], degree=case["degree"],
                                n_paths_oos=case["n_oos"])
    return st


# Fields of a result that hold device times, not results.
TIMES = ("kernel_ms", "select_ms", "sim_ms", "regress_ms", "oos_ms", "update_ms")


def _numbers(r):
    return {k: v for k, v in r.items() if k not in TIMES}


def run(st):
    c, kind = st["case"], st["case"]["kind"]
    if kind == "multi":
        st["call"]()
        return [_numbers(r) for r in st["call"].results()]
    if kind == "autograd":
        m = st["m"]
        S0 = torch.tensor(m["S0"], dtype=torch.float64, requires_grad=True)
        v0 = torch.tensor(m["v0"], dtype=torch.float64, requires_grad=True)
        price = mc.PathwisePrice.apply(S0, v0, st["ctx"], st["model"], st["payoff"], c["n_paths"],
                                       c["n_steps"], st["key"])
        price.backward()
        return {"price": price.detach(), "d_S0": S0.grad, "d_v0": v0.grad}
    if kind == "cv_train":
        w, log = mc.mc_cv_train(st["ctx"], st["model"], st["payoff"], c["n_train"], c["n_steps"],
                                st["key"], st["weights"], steps=c["adam_steps"], batch=c["batch"],
                                hedge_every=c["hedge_every"], prec=PRECS[c["prec"]], **ADAM)
        return {"weights": w, "loss": log}
    if kind == "risk":
        return _numbers(mc.mc_risk(st["ctx"], st["model"], PORTFOLIO[0], PORTFOLIO[1], 0.99,
                                   c["n_paths"], c["n_steps"], st["key"], mu=st["m"]["mu"],
                                   opts=st["opts"]))
    if kind == "qmc":
        r = _numbers(mc.mc_price_qmc(st["ctx"], st["model"], st["payoff"], c["n_paths"],
                                     c["n_steps"], st["key"], c["replicates"], st["opts"]))
        r["replicate_price"] = np.array(r["replicate_price"], np.float32)
        r["replicate_geo"] = np.array(r["replicate_geo"], np.float32)
        return r
    if kind == "lsm":
        return _numbers(mc.mc_price_lsm(st["ctx"], st["model"], st["spec"], c["n_paths"], st["key"]))
    return _numbers(mc.mc_price(st["ctx"], st["model"], st["payoff"], c["n_paths"], c["n_steps"],
                                st["key"], st["opts"]))


# ----------------------------------------------------------------- work ----
# Arithmetic of one normal: a quarter of a Philox block (20 products of two
# halves, 40 xors, 20 key additions) and its share of Box-Muller (log, square
# root, sine, cosine, four multiply-adds for two normals).
NORMAL = (40 + 40 + 20) / 4 + 4


def work(case):
    k, n, N = case["kind"], case.get("n_steps", 1), case.get("n_paths", 0)
    if k == "gbm":
        f = N * n * (NORMAL + 6)
        if case["greeks"] == "fd":
            f += 4 * N * n * (NORMAL + 6)      # an up and a down run for each of two greeks
        b = 1e3
    elif k == "multi":
        f, b = N * n * (NORMAL + 7), 1e3
    elif k in ("heston", "autograd"):
        per = 2 * NORMAL + 18
        f = N * n * (per + (14 if k == "autograd" or case["greeks"] else 0))
        b = 1e3
    elif k == "cv_price":
        f = N * n * (2 * NORMAL + 18) + N * -(-n // case["hedge_every"]) * (2 * 4480 + 6 * 128)
        b = 4545 * 4
    elif k == "cv_train":
        items = case["batch"] * -(-n // case["hedge_every"])
        f = case["n_train"] * n * (2 * NORMAL + 18) + case["adam_steps"] * items * 3 * (2 * 4480 + 768)
        b = 4545 * 8
    elif k in ("basket", "risk"):
        d = case["d"]
        f, b = N * n * d * NORMAL + N * d * (d + 1) + N * d * 12, d * d * 8
    elif k == "qmc":
        d = case["d"]
        f, b = case["replicates"] * N * (n * d * 12 + d * (d + 1) + d * 12), d * d * 8
    else:
        d, M, No = case["d"], case["n_dates"], case["n_oos"]
        nf = 2 + case["degree"] * d
        f = (N + No) * M * d * (NORMAL + 6) + N * (M - 1) * (nf + 1) * (nf + 2) + (N + No) * M * 4 * nf
        b = 1e4
    return {"bytes": float(b), "flops": float(f)}


# ---------------------------------------------------------------- exact ----
DEV = "cuda" if torch.cuda.is_available() else "cpu"
M32 = 0xFFFFFFFF
F64 = torch.float64


def _words(key, tag, path, j):
    """Philox4x32-10 block j of each path (j a number, or a tensor that
    broadcasts with path): four int64 tensors of 32-bit words."""
    c0 = torch.full_like(path, j) if isinstance(j, int) else j
    c1, c2 = path & M32, path >> 32
    c3 = torch.full_like(path, tag)
    k0, k1 = key & M32, key >> 32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57       # modulo 2^64
        c0, c1, c2, c3 = (((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32,
                          ((p0 >> 32) & M32) ^ c3 ^ k1, p0 & M32)
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _unit(w):
    return (2 * (w >> 9) + 1).to(F64) * 2.0 ** -24


def _box_muller(w):
    out = []
    for a, b in ((w[0], w[1]), (w[2], w[3])):
        r = torch.sqrt(-2.0 * torch.log(_unit(a)))
        ang = 2.0 * math.pi * _unit(b)
        out += [r * torch.cos(ang), r * torch.sin(ang)]
    return out


class _Normals:
    """Normals of a set of paths in index order."""

    def __init__(self, key, tag, path):
        self.key, self.tag, self.path, self.j, self.z = key, tag, path, -1, None

    def __call__(self, k):
        if k // 4 != self.j:
            self.j = k // 4
            self.z = _box_muller(_words(self.key, self.tag, self.path, self.j))
        return self.z[k % 4]


def _chunks(N, most):
    for a in range(0, N, most):
        yield torch.arange(a, min(N, a + most), dtype=torch.int64, device=DEV)


class _Sums:
    """Means and covariances of columns over chunks of paths."""

    def __init__(self):
        self.n, self.mean, self.co = 0, None, None

    def add(self, *cols):
        y = torch.stack([c.expand(cols[0].shape) for c in cols])
        n, mean = y.shape[1], y.mean(1)
        dev = y - mean[:, None]
        co = dev @ dev.T
        if not self.n:
            self.n, self.mean, self.co = n, mean, co
            return
        d = mean - self.mean
        t = self.n + n
        self.co = self.co + co + torch.outer(d, d) * (self.n * n / t)
        self.mean = self.mean + d * (n / t)
        self.n = t

    def cov(self, a, b):
        return float(self.co[a, b]) / (self.n - 1)

    def of(self, c):
        return float(self.mean[c]), math.sqrt(self.cov(c, c) / self.n)


def _result(price, se, var, plain=None, delta=(0.0, 0.0), vega=(0.0, 0.0), beta=0.0, vrf=1.0):
    p = plain or (price, se)
    return dict(price=price, std_err=se, variance=var, delta=delta[0], delta_se=delta[1],
                vega=vega[0], vega_se=vega[1], plain_price=p[0], plain_std_err=p[1], cv_beta=beta,
                vrf=vrf, n_paths=None, n_nonfinite=None, cv_fallback=None, greeks_method=None)


def _pos(x):
    return torch.clamp(x, min=0.0)


def _gbm_paths(m, n, path, key, payoffs, S0=None, sigma=None, bridge=False):
    """Running functionals of log-Euler paths: S_T, mean S, mean ln S, alive flags, W_T and the
    Asian's d(sum S)/d sigma."""
    S0 = m["S0"] if S0 is None else S0
    sg = m["sigma"] if sigma is None else sigma
    dt = m["T"] / n
    drift, vol, lnB = (m["rate"] - 0.5 * sg * sg) * dt, sg * math.sqrt(dt), math.log(m["B"] / S0)
    Z = _Normals(key, 0, path)
    x = torch.zeros(path.shape, dtype=F64, device=DEV)
    sE, sx, W, dV = x.clone(), x.clone(), x.clone(), x.clone()
    alive = torch.ones(path.shape, dtype=torch.bool, device=DEV)
    alive_bb = alive.clone()
    wb = None
    for i in range(n):
        z = Z(i)
        xp = x
        x = x + drift + vol * z
        W = W + z * math.sqrt(dt)
        alive = alive & (x < lnB)
        if bridge:
            if i % 4 == 0:
                wb = _words(key, 5, path, i // 4)
            top = 0.5 * (xp + x + torch.sqrt((xp - x) ** 2 - 2.0 * dt * sg * sg *
                                             torch.log(_unit(wb[i % 4]))))
            alive_bb = alive_bb & (top < lnB)
        if "asian" in payoffs:
            E = torch.exp(x)
            sE = sE + E
            sx = sx + x
            dV = dV + E * (W - sg * dt * (i + 1))
    return dict(ST=S0 * torch.exp(x), A=S0 * sE / n, G=S0 * torch.exp(sx / n), alive=alive,
                alive_bb=alive_bb, W=W, dV=S0 * dV / n)


def _geo_mean(m, n):
    S0, K, r, sg, T = m["S0"], m["K"], m["rate"], m["sigma"], m["T"]
    mu = math.log(S0) + (r - 0.5 * sg * sg) * T * (n + 1) / (2 * n)
    s2 = sg * sg * T * (n + 1) * (2 * n + 1) / (6 * n * n)
    N = lambda q: 0.5 * math.erfc(-q / math.sqrt(2.0))
    s = math.sqrt(s2)
    d2 = (mu - math.log(K)) / s
    return math.exp(-r * T) * (math.exp(mu + 0.5 * s2) * N(d2 + s) - K * N(d2))


def _payoff_gbm(kind, p, K, disc):
    if kind == "asian":
        return disc * _pos(p["A"] - K)
    call = disc * _pos(p["ST"] - K)
    return call if kind == "euro" else call * (p["alive"] if kind == "uo" else p["alive_bb"])


def _with_cv(s, a, g, CG):
    beta = s.cov(a, g) / s.cov(g, g)
    price = float(s.mean[a]) - beta * (float(s.mean[g]) - CG)
    var = s.cov(a, a) - 2 * beta * s.cov(a, g) + beta * beta * s.cov(g, g)
    return _result(price, math.sqrt(var / s.n), var, plain=s.of(a), beta=beta, vrf=s.cov(a, a) / var)


def _exact_gbm(case, m):
    K, disc, n = m["K"], math.exp(-m["rate"] * m["T"]), case["n_steps"]
    kind, fd, h = case["payoff"], case["greeks"] == "fd", 1e-3
    s = _Sums()
    for path in _chunks(case["n_paths"], 1 << 20):
        go = lambda **k: _payoff_gbm(kind, _gbm_paths(m, n, path, m["key"], (kind,),
                                                      bridge=kind == "bridge", **k), K, disc)
        p = _gbm_paths(m, n, path, m["key"], (kind,), bridge=kind == "bridge")
        cols = [_payoff_gbm(kind, p, K, disc)]
        if case["cv"]:
            cols.append(disc * _pos(p["G"] - K))
        if fd:
            S0, sg = m["S0"], m["sigma"]
            cols.append((go(S0=S0 * (1 + h)) - go(S0=S0 * (1 - h))) / (2 * h * S0))
            cols.append((go(sigma=sg * (1 + h)) - go(sigma=sg * (1 - h))) / (2 * h * sg))
        elif case["greeks"]:
            x = p["A"] if kind == "asian" else p["ST"]
            itm = (x > K).to(F64) * disc
            cols.append(itm * x / m["S0"])
            cols.append(itm * (p["dV"] if kind == "asian" else x * (p["W"] - m["sigma"] * m["T"])))
        s.add(*cols)
    if case["cv"]:
        return _with_cv(s, 0, 1, _geo_mean(m, n))
    g = (s.of(1), s.of(2)) if case["greeks"] else ((0.0, 0.0), (0.0, 0.0))
    return _result(*s.of(0), s.cov(0, 0), delta=g[0], vega=g[1])


def _exact_multi(case, m):
    K, disc, n = m["K"], math.exp(-m["rate"] * m["T"]), case["n_steps"]
    s = _Sums()
    for path in _chunks(case["n_paths"], 1 << 22):
        p = _gbm_paths(m, n, path, m["key"], ("asian",))
        s.add(disc * _pos(p["A"] - K), disc * _pos(p["G"] - K),
              disc * _pos(p["ST"] - K) * p["alive"])
    return [_with_cv(s, 0, 1, _geo_mean(m, n)), _result(*s.of(2), s.cov(2, 2)),
            _result(*s.of(1), s.cov(1, 1))]


def _heston_steps(m, n, path, key, tag, each):
    """Full-truncation Euler on (ln S/S0, v); each(i, before, z1, zs, vp, sq, x, v)."""
    dt = m["T"] / n
    Z = _Normals(key, tag, path)
    x = torch.zeros(path.shape, dtype=F64, device=DEV)
    v = torch.full(path.shape, m["v0"], dtype=F64, device=DEV)
    rc = math.sqrt(1.0 - m["rho"] ** 2)
    for i in range(n):
        z1, z2 = Z(2 * i), Z(2 * i + 1)
        vp = _pos(v)
        sq = torch.sqrt(vp * dt)
        zs = m["rho"] * z1 + rc * z2
        x = x + (m["rate"] - 0.5 * vp) * dt + sq * zs
        vb = v
        v = v + m["kappa"] * (m["theta"] - vp) * dt + m["xi"] * sq * z1
        each(i, vb, z1, zs, vp, sq, x, v)
    return x, v


def _exact_heston(case, m, greeks):
    n, K, S0, disc, dt = (case["n_steps"], m["K"], m["S0"], math.exp(-m["rate"] * m["T"]),
                          m["T"] / case["n_steps"])
    asian = case["payoff"] == "asian"
    s = _Sums()
    for path in _chunks(case["n_paths"], 1 << 21):
        z = torch.zeros(path.shape, dtype=F64, device=DEV)
        a = dict(E=z, Ed=z, dx=z, dv=z + 1.0)

        def each(i, v, z1, zs, vp, sq, x, _):
            up = v > 0
            dvp = torch.where(up, a["dv"], z)
            dsq = torch.where(up, 0.5 * dt * dvp / torch.where(up, sq, z + 1.0), z)
            a["dx"] = a["dx"] - 0.5 * dt * dvp + dsq * zs
            a["dv"] = a["dv"] - m["kappa"] * dt * dvp + m["xi"] * dsq * z1
            if asian:
                E = torch.exp(x)
                a["E"] = a["E"] + E
                a["Ed"] = a["Ed"] + E * a["dx"]

        x, _ = _heston_steps(m, n, path, m["key"], 0, each)
        S = S0 * a["E"] / n if asian else S0 * torch.exp(x)
        dv0 = S0 * a["Ed"] / n if asian else S * a["dx"]
        itm = (S > K).to(F64) * disc
        s.add(disc * _pos(S - K), itm * S / S0, itm * dv0)
    return s if greeks is None else _result(
        *s.of(0), s.cov(0, 0), delta=s.of(1) if greeks else (0.0, 0.0),
        # The sample spread of d/dv0 is set by the few paths that pass near
        # v = 0 (its derivative has no bound there): it has no 64-bit value
        # that a path of another rounding could be held to.
        vega=(s.of(2)[0], None) if greeks else (0.0, 0.0))


def _cv_segments(m, n, every, path, tag, each_segment):
    """Hedge segments of Heston paths: features at each opening date and the
    discounted price change over it; returns the discounted Asian payoff."""
    z = torch.zeros(path.shape, dtype=F64, device=DEV)
    r, S0, K, dt = m["rate"], m["S0"], m["K"], m["T"] / n
    a = dict(sum=z, open=None, phi=None)

    def features(i, x, v):
        mean = S0 * a["sum"] / i if i else z + S0
        return torch.stack([z + i / n, x + math.log(S0 / K), v / m["theta"], mean / K - 1.0], 1)

    a["phi"], a["open"] = features(0, z, z + m["v0"]), z + S0

    def each(i, vb, z1, zs, vp, sq, x, v):
        S = S0 * torch.exp(x)
        a["sum"] = a["sum"] + S / S0
        if (i + 1) % every == 0 or i + 1 == n:
            St = S * math.exp(-r * dt * (i + 1))
            each_segment(a["phi"], St - a["open"])
            if i + 1 < n:
                a["phi"], a["open"] = features(i + 1, x, v), St

    _heston_steps(m, n, path, m["key"], tag, each)
    return math.exp(-r * m["T"]) * _pos(S0 * a["sum"] / n - K)


def _net(w, phi):
    W1, b1, W2 = w[:256].view(64, 4), w[256:320], w[320:4416].view(64, 64)
    b2, W3, b3 = w[4416:4480], w[4480:4544], w[4544]
    return torch.tanh(torch.tanh(phi @ W1.T + b1) @ W2.T + b2) @ W3 + b3


def _exact_cv_price(case, m, seed):
    w = torch.from_numpy(_hedge_weights(m, seed)).to(DEV, F64)
    s = _Sums()
    for path in _chunks(case["n_paths"], 1 << 19):
        H = [torch.zeros(path.shape, dtype=F64, device=DEV)]

        def seg(phi, dS):
            H[0] = H[0] + _net(w, phi) * dS

        pay = _cv_segments(m, case["n_steps"], case["hedge_every"], path, 0, seg)
        s.add(pay, pay - H[0])
    var = s.cov(1, 1)
    return _result(*s.of(1), var, plain=s.of(0), beta=1.0, vrf=s.cov(0, 0) / var)


def _exact_cv_train(case, m, seed):
    B, segs, pays = case["batch"], [], None
    path = torch.arange(case["n_train"], dtype=torch.int64, device=DEV)
    pays = _cv_segments(m, case["n_steps"], case["hedge_every"], path, 2,
                        lambda phi, dS: segs.append((phi, dS)))
    w = torch.from_numpy(_glorot(seed)).to(DEV, F64)
    mom, vel = torch.zeros_like(w), torch.zeros_like(w)
    b1, b2, log = ADAM["beta1"], ADAM["beta2"], []
    for t in range(case["adam_steps"]):
        a = (t % (case["n_train"] // B)) * B
        wt = w.clone().requires_grad_(True)
        H = sum(_net(wt, phi[a:a + B]) * dS[a:a + B] for phi, dS in segs)
        Y = pays[a:a + B] - H
        loss = ((Y - Y.mean()) ** 2).mean()
        loss.backward()
        g = wt.grad
        log.append(float(loss.detach()))
        mom = b1 * mom + (1 - b1) * g
        vel = b2 * vel + (1 - b2) * g * g
        w = w - ADAM["lr"] * (mom / (1 - b1 ** (t + 1))) / (torch.sqrt(vel / (1 - b2 ** (t + 1))) +
                                                          ADAM["eps"])
    return {"weights": w, "loss": np.array(log)}


def _correlated(m, d, n):
    L = np.linalg.cholesky(np.asarray(m["corr"], np.float64))
    Ls = np.asarray(m["sigma"])[:, None] * math.sqrt(m["T"] / n) * L
    return torch.from_numpy(Ls).to(DEV)


def _basket_logs(m, case, path, normals, drift):
    """ln(S_a,T / S0_a) of each path: the increments L Z summed over the steps."""
    d, n = case["d"], case["n_steps"]
    J = d // 4
    Z = torch.zeros((J, 4, path.numel()), dtype=F64, device=DEV)
    for i in range(n):
        q = normals(torch.arange(i * J, (i + 1) * J, dtype=torch.int64, device=DEV)[:, None])
        for t in range(4):
            Z[:, t] += q[t]
    sg = torch.tensor(m["sigma"], dtype=F64, device=DEV)
    mu = torch.tensor(drift, dtype=F64, device=DEV)
    return Z.view(d, -1).T @ _correlated(m, d, n).T + (mu - 0.5 * sg * sg) * m["T"]


def _exact_basket(case, m):
    d, S0, K, disc = case["d"], m["S0"][0], m["K"], math.exp(-m["rate"] * m["T"])
    s = _Sums()
    for path in _chunks(case["n_paths"], 1 << 18):
        x = _basket_logs(m, case, path,
                         lambda j: _box_muller(_words(m["key"], 0, path[None, :], j)), [m["rate"]] * d)
        E = torch.exp(x)
        A = S0 * E.mean(1)
        s.add(disc * _pos(A - K), (A > K).to(F64) * disc * E[:, 0] / d)
    return _result(*s.of(0), s.cov(0, 0), delta=s.of(1))


def _exact_risk(case, m):
    d, S0, T, r = case["d"], m["S0"][0], m["T"], m["rate"]
    mult, qty = PORTFOLIO
    N = lambda q: 0.5 * math.erfc(-q / math.sqrt(2.0))
    V0 = 0.0
    for sg in m["sigma"]:
        for k, q in zip(mult, qty):
            st = sg * math.sqrt(T)
            d1 = (-math.log(k) + (r + 0.5 * sg * sg) * T) / st
            V0 += q * (S0 * N(d1) - k * S0 * math.exp(-r * T) * N(d1 - st))
    pnl = []
    for path in _chunks(case["n_paths"], 1 << 18):
        E = torch.exp(_basket_logs(m, case, path,
                                   lambda j: _box_muller(_words(m["key"], 0, path[None, :], j)), m["mu"]))
        v = sum(q * _pos(E - k) for k, q in zip(mult, qty))
        pnl.append(S0 * v.sum(1) - V0)
    pnl = torch.sort(torch.cat(pnl)).values
    n = pnl.numel()
    k = int(math.floor(n * (1.0 - 0.99))) + 1
    cut = float(pnl[k - 1])
    tail = pnl[pnl < pnl[k - 1]]
    return dict(var=-cut, cvar=-float(tail.mean()), quantile_pnl=cut, pnl_mean=float(pnl.mean()),
                pnl_std_err=float(pnl.std(unbiased=True)) / math.sqrt(n), premium=V0, k=None,
                n_tail=None, n_paths=None)


def _sobol_directions(dims):
    """Direction words [dims][32]: primitive polynomials by degree and bit
    pattern, first direction integers from SplitMix64, then the recursion."""
    def mix(x):
        U = (1 << 64) - 1
        x = (x + 0x9E3779B97F4A7C15) & U
        x = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & U
        x = ((x ^ (x >> 27)) * 0x94D049BB133111EB) & U
        return x ^ (x >> 31)

    def order_is_full(p, s):
        x, n = 1, 0
        while True:
            x <<= 1
            if x >> s & 1:
                x ^= p
            n += 1
            if x == 1:
                return n == (1 << s) - 1
            if x == 0 or n > 1 << s:
                return False

    V = [[1 << (31 - b) for b in range(32)]]
    s = 1
    while len(V) < dims:
        for p in range((1 << s) | 1, 2 << s, 2):
            if len(V) == dims or not order_is_full(p, s):
                continue
            j = len(V)
            mi = [0] + [2 * (mix(64 * j + i) % (1 << (i - 1))) + 1 for i in range(1, s + 1)]
            for i in range(s + 1, 33):
                v = mi[i - s] ^ (mi[i - s] << s)
                for k in range(1, s):
                    if p >> (s - k) & 1:
                        v ^= mi[i - k] << k
                mi.append(v)
            V.append([(mi[b + 1] << (31 - b)) & M32 for b in range(32)])
        s += 1
    return V


def _exact_qmc(case, m):
    d, n, K, disc = case["d"], case["n_steps"], m["K"], math.exp(-m["rate"] * m["T"])
    V = _sobol_directions(n * d)
    path = torch.arange(case["n_paths"], dtype=torch.int64, device=DEV)
    words = torch.zeros((n * d, case["n_paths"]), dtype=torch.int64, device=DEV)
    V = torch.tensor(V, dtype=torch.int64, device=DEV)
    for b in range(32):
        if case["n_paths"] >> b:
            words ^= torch.where((path >> b & 1) == 1, V[:, b:b + 1], 0)
    one = torch.arange(case["replicates"], dtype=torch.int64, device=DEV)[:, None]
    j = torch.arange(n * d // 4, dtype=torch.int64, device=DEV)[None, :]
    shift = torch.stack(torch.broadcast_tensors(*_words(m["key"], 6, one, j)), 2)
    shift = shift.reshape(case["replicates"], n * d, 1)
    prices, geos = [], []
    for rep in range(case["replicates"]):
        x = _basket_logs(m, case, path, lambda j: _box_muller(
            [(words ^ shift[rep])[j[:, 0] * 4 + t] for t in range(4)]), [m["rate"]] * d)
        S0 = m["S0"][0]
        prices.append(float((disc * _pos(S0 * torch.exp(x).mean(1) - K)).mean()))
        geos.append(float((disc * _pos(S0 * torch.exp(x.mean(1)) - K)).mean()))
    p, g, R = np.array(prices), np.array(geos), case["replicates"]
    return dict(price=float(p.mean()), std_err=float(p.std(ddof=1)) / math.sqrt(R),
                geo_price=float(g.mean()), geo_std_err=float(g.std(ddof=1)) / math.sqrt(R),
                n_replicates=None, n_points=None, replicate_price=p, replicate_geo=g)


def _lsm_paths(case, m, N, tag):
    """y = S/K at each date, a list of [N, d] tensors."""
    d, M = case["d"], case["n_dates"]
    n = M * case["steps_per_date"]
    Ls = _correlated(m, d, n)
    sg = torch.tensor(m["sigma"], dtype=F64, device=DEV)
    drift = (m["rate"] - m["q"] - 0.5 * sg * sg) * (m["T"] / n)
    x = torch.log(torch.tensor(m["S0"], dtype=F64, device=DEV) / m["K"]).repeat(N, 1)
    Z = _Normals(m["key"], tag, torch.arange(N, dtype=torch.int64, device=DEV))
    ys = []
    for i in range(n):
        z = torch.stack([Z(i * d + a) for a in range(d)], 1)
        x = x + drift + z @ Ls.T
        if (i + 1) % case["steps_per_date"] == 0:
            ys.append(torch.exp(x))
    return ys


def _lsm_features(case, y, f):
    d, cols = case["d"], [torch.ones_like(f)]
    cols += [y[:, a] for a in range(d)]
    if case["degree"] >= 2:
        cols += [y[:, a] * y[:, b] for a in range(d) for b in range(a, d)]
    if case["payoff"] == "max_call" and d >= 2:
        cols.append(f)
    return torch.stack(cols, 1)


def _exact_lsm(case, m):
    M, K = case["n_dates"], m["K"]
    dK = [K * math.exp(-m["rate"] * m["T"] * j / M) for j in range(M + 1)]
    pay = ((lambda y: _pos(y.max(1).values - 1.0)) if case["payoff"] == "max_call"
           else (lambda y: _pos(1.0 - y.mean(1))))
    ys = _lsm_paths(case, m, case["n_paths"], 0)
    C = dK[M] * pay(ys[-1])
    mean_se = lambda v: (float(v.mean()), float(v.std(unbiased=True)) / math.sqrt(v.numel()))
    euro = mean_se(C)
    betas = [None] * M
    for j in range(M - 1, 0, -1):
        f = pay(ys[j - 1])
        itm = f > 0
        X = _lsm_features(case, ys[j - 1][itm], f[itm])
        beta = torch.linalg.solve(X.T @ X, X.T @ C[itm])
        ex = dK[j] * f[itm] >= X @ beta
        C[itm] = torch.where(ex, dK[j] * f[itm], C[itm])
        betas[j - 1] = beta
    price = mean_se(C)
    v = None
    live = torch.ones(case["n_oos"], dtype=torch.bool, device=DEV)
    v = torch.zeros(case["n_oos"], dtype=F64, device=DEV)
    for j, y in enumerate(_lsm_paths(case, m, case["n_oos"], 7), 1):
        f = pay(y)
        stop = live & (f > 0)
        if j < M:
            stop = stop & (dK[j] * f >= _lsm_features(case, y, f) @ betas[j - 1])
        v = torch.where(stop, dK[j] * f, v)
        live = live & ~stop
    oos = mean_se(v)
    nf = betas[0].numel()
    rows = [b.cpu().numpy() if b is not None else np.full(nf, np.nan) for b in betas]
    return dict(price=price[0], std_err=price[1], price_oos=oos[0], std_err_oos=oos[1],
                european=euro[0], european_se=euro[1], n_features=None, beta=np.array(rows),
                beta_valid=None, n_itm=None, n_paths=None, n_paths_oos=None)


def exact(case, seed):
    m, kind = _market(case, seed), case["kind"]
    with torch.no_grad() if kind != "cv_train" else torch.enable_grad():
        if kind == "gbm":
            return _exact_gbm(case, m)
        if kind == "multi":
            return _exact_multi(case, m)
        if kind == "heston":
            return _exact_heston(case, m, case["greeks"])
        if kind == "autograd":
            s = _exact_heston(case, m, None)
            return {"price": s.of(0)[0], "d_S0": s.of(1)[0], "d_v0": s.of(2)[0]}
        if kind == "cv_price":
            return _exact_cv_price(case, m, seed)
        if kind == "cv_train":
            return _exact_cv_train(case, m, seed)
        if kind == "basket":
            return _exact_basket(case, m)
        if kind == "risk":
            return _exact_risk(case, m)
        if kind == "qmc":
            return _exact_qmc(case, m)
        return _exact_lsm(case, m)
