"""GPU tests of the kernels' branches at the sizes where they can go wrong:
remainders of a Philox block, path indices that straddle 2^32, functional sets
of their own, the edges of tiles. Each is held to the FP64 oracle or to the
general path."""
import ctypes as C
import math

import numpy as np
import pytest

import oracle
import paper_1906_02818_amd as mc
import synth
from paper_1906_02818_amd import _abi
from lsm_basis import MAXC, PUT

pytestmark = pytest.mark.gpu

SEED = synth.SEED
G = dict(S0=100.0, r=0.03, sigma=0.25, T=1.0, K=100.0, B=125.0)


@pytest.fixture(scope="module")
def ctx():
    c = mc.mc_create(0)
    yield c
    c.close()


def gbm():
    return mc.Model(kind=mc.MC_GBM, S0=G["S0"], r=G["r"], T=G["T"], sigma=G["sigma"])


def ora(n, N, path0=0):
    return oracle.gbm(G["S0"], G["r"], G["sigma"], G["T"], G["K"], G["B"], n, N, SEED, path0=path0)


GBM_SETS = [(mc.MC_EURO_CALL, 0, 0), (mc.MC_EURO_CALL, 3, 0), (mc.MC_ASIAN_ARITH_CALL, 0, 1),
            (mc.MC_ASIAN_ARITH_CALL, 3, 1), (mc.MC_ASIAN_GEO_CALL, 0, 2),
            (mc.MC_UO_BARRIER_CALL, 0, 3), (mc.MC_UO_BRIDGE_CALL, 0, 9)]


@pytest.mark.parametrize("prec", [mc.MC_FP64, mc.MC_FP32])
@pytest.mark.parametrize("N,n", [(2, 1), (257, 3), (1000, 6), (4099, 64)])
def test_each_functional_set_prices_like_the_oracle(ctx, prec, N, n):
    # Without per-path rows a call runs on the smallest set of functionals
    # that covers its payoff. FP64: the oracle's own precision; FP32: the
    # 2e-5 of every FP32 price, on the scale of S0 (few paths may all be out
    # of the money or sit at the strike).
    o = ora(n, N)
    for kind, greeks, col in GBM_SETS:
        print("set", kind, greeks, prec, N, n, flush=True)
        r = mc.mc_price(ctx, gbm(), mc.Payoff(kind, G["K"], B=G["B"]), N, n, SEED,
                        mc.Options(prec=prec, greeks=greeks))
        y = o[:, col].copy()
        slack = 0.0
        if kind in (mc.MC_UO_BARRIER_CALL, mc.MC_UO_BRIDGE_CALL):
            marg = np.abs(o[:, 10 if kind == mc.MC_UO_BARRIER_CALL else 11])
            slack = G["B"] * np.mean(marg < (1e-12 if prec == mc.MC_FP64 else 2e-5))
        tol = 1e-12 if prec == mc.MC_FP64 else 2e-5
        assert abs(r["price"] - y.mean()) <= tol * G["S0"] + slack
        if greeks:
            g = o[:, [4, 5]] if kind == mc.MC_EURO_CALL else o[:, [6, 7]]
            at_kink = np.mean(np.abs(y) < (1e-11 if prec == mc.MC_FP64 else 1e-3) * (y != 0))
            assert abs(r["delta"] - g[:, 0].mean()) <= tol * 10 + 2 * at_kink
            assert abs(r["vega"] - g[:, 1].mean()) <= tol * 1000 + 200 * at_kink


@pytest.mark.parametrize("prec", [mc.MC_FP64, mc.MC_FP32])
@pytest.mark.parametrize("offset,n", [((1 << 32) - 1, 1), ((1 << 32) - 65, 4), ((1 << 33) - 64, 7),
                                      ((1 << 32) - 200, 5)])
def test_paths_across_a_multiple_of_2p32(ctx, prec, offset, n):
    # A wave whose paths straddle a multiple of 2^32 takes two passes.
    N = 323
    print("straddle", prec, offset, n, flush=True)
    r = mc.mc_price(ctx, gbm(), mc.Payoff(mc.MC_ASIAN_ARITH_CALL, G["K"]), N, n, SEED,
                    mc.Options(prec=prec, path_offset=offset, path_values=True))
    o = ora(n, N, path0=offset)
    j = r["path_channels"].index("asian")
    tol = 1e-11 if prec == mc.MC_FP64 else 3e-4
    np.testing.assert_allclose(r["path_values"][:, j], o[:, 1], rtol=tol, atol=tol)


@pytest.mark.parametrize("path,k0", [(0, 0), (5, 3), ((1 << 40) + 1, 12345)])
def test_fp64_normals_to_rounding(ctx, path, k0):
    # 2^17 normals against the oracle's: a few roundings of values below 5.8.
    z = mc.mc_normals(ctx, SEED, 0, path, k0, 1 << 17, mc.MC_FP64)
    ref = oracle.normals(SEED, 0, path, k0, 1 << 17)
    assert np.max(np.abs(z - ref)) < 6e-15


# ------------------------------------------------------------- basket ----
def _bf16(x):
    u = np.ascontiguousarray(x, np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


def _rounded(x, prec):
    """x as the operand of a product of this precision (float64 result)."""
    if prec == mc.MC_FP32:
        return np.asarray(x, np.float32).astype(np.float64)
    if prec == mc.MC_FP16_GEMM:
        return np.asarray(np.asarray(x, np.float32), np.float16).astype(np.float64)
    return _bf16(x)


@pytest.mark.parametrize("prec", [mc.MC_FP32, mc.MC_BF16_GEMM, mc.MC_FP16_GEMM, mc.MC_BF16X2_GEMM])
@pytest.mark.parametrize("d,N,n,offset", [(16, 2, 1, 0), (16, 4099, 3, 5), (64, 63, 2, 0),
                                          (80, 65, 3, (1 << 32) - 33), (128, 200, 1, 0),
                                          (144, 129, 2, 7), (256, 64, 5, 0)])
def test_basket_tiles_and_forms(ctx, prec, d, N, n, offset):
    # Every wave layout, partial tiles, odd and single steps, all operand
    # forms: the log-prices of a model that rounds each step's normals and L'
    # as the form's operands and does everything else in 64 bits. The kernel
    # adds FP32 rounding (1e-6 of a price); a normal within FP32 error of a
    # rounding boundary (one in 2^14) may round to the other side.
    print("basket tiles", prec, d, N, n, offset, flush=True)
    sigma, corr, _ = synth.basket_market(d)
    rng = np.random.default_rng(d + n)
    S0 = 80.0 + 40.0 * rng.random(d)
    w = rng.random(d) / d
    K, r_, T = 40.0, 0.05, 1.0
    r = mc.mc_price(ctx, mc.Model(kind=mc.MC_GBM_BASKET, S0=S0, r=r_, T=T, sigma=sigma, corr=corr),
                    mc.Payoff(mc.MC_BASKET_CALL, K, weights=w), N, n, SEED,
                    mc.Options(prec=prec, path_offset=offset, path_values=True))
    L = np.linalg.cholesky(corr) * (sigma * np.sqrt(T / n) / np.log(2.0))[:, None]
    Lr = _rounded(L, prec)
    if prec == mc.MC_BF16X2_GEMM:
        Lr = Lr + _bf16(L - Lr)
    keep = np.arange(N) if N <= 300 else np.unique(np.r_[0:70, N - 70:N])
    x = np.empty((keep.size, d))
    for row, p in enumerate(keep):
        z = oracle.normals(SEED, 0, offset + int(p), 0, n * d).reshape(n, d)
        x[row] = Lr @ _rounded(z, prec).sum(0)
    E = 2.0 ** (x + (r_ - 0.5 * sigma * sigma) * T / np.log(2.0))
    basket = (E * S0 * w).sum(1)
    ref = np.exp(-r_ * T) * np.maximum(basket - K, 0.0)
    err = np.abs(r["path_values"][keep, 0] - ref)
    tol = 4e-6 * (S0 * w).sum()
    flips = 0.0 if prec == mc.MC_FP32 else n * d * 2.0 ** -14
    assert np.mean(err > tol) <= 2.0 * flips + (4.0 / keep.size if flips else 0.0)
    assert err.max() <= (tol if prec == mc.MC_FP32 else 2e-2 * (S0 * w).sum())
    assert r["n_paths"] == N and r["n_nonfinite"] == 0


@pytest.mark.parametrize("offset,N", [(0, 64), (0, 1), (1, 200), (61, 131), ((1 << 20) - 3, 70),
                                      ((1 << 32) - 90, 90)])
def test_sobol_points_at_any_offset(ctx, offset, N):
    # Points whose tile starts at, or between, multiples of 64.
    if N == 1:
        N = 2
    d, n = 16, 2
    print("sobol offset", offset, N, flush=True)
    sigma, corr, _ = synth.basket_market(d)
    S0, w = np.full(d, 100.0), np.full(d, 1.0 / d)
    model = mc.Model(kind=mc.MC_GBM_BASKET, S0=S0, r=0.05, T=1.0, sigma=sigma, corr=corr)
    r = mc.mc_price_qmc(ctx, model, mc.Payoff(mc.MC_BASKET_CALL, 90.0), N, n, SEED, 1,
                        mc.Options(prec=mc.MC_FP32, path_offset=offset, path_values=True))
    o = oracle.basket_qmc(S0, sigma, oracle.cholesky(corr), w, 0.05, 1.0, 90.0, n, N, SEED,
                          0, path0=offset)
    np.testing.assert_allclose(r["path_values"][:, 0], o[:, 0], rtol=1e-4, atol=1e-4)


# ------------------------------------------------------------- Heston ----
H = synth.HESTON


def heston():
    return mc.Model(kind=mc.MC_HESTON, S0=H["S0"], r=H["r"], T=H["T"], v0=H["v0"],
                    kappa=H["kappa"], theta=H["theta"], xi=H["xi"], rho=H["rho"])


@pytest.mark.parametrize("kind", [mc.MC_ASIAN_ARITH_CALL, mc.MC_EURO_CALL])
@pytest.mark.parametrize("N,n,offset", [(2, 1, 0), (257, 2, 3), (1000, 17, (1 << 32) - 500),
                                        (300, 259, 0)])
def test_pathwise_greeks_equal_the_adjoint(ctx, kind, N, n, offset):
    # The same FP32 state and step derivatives, multiplied forward instead of
    # backward in FP64: equal to the rounding of at most 2 n products, on the
    # scale of the largest path (products of factors up to 1e3 near v = 0).
    print("pathwise = adjoint", kind, N, n, offset, flush=True)
    f = mc.Payoff(kind, H["K"])
    a = mc.mc_greeks_adjoint(ctx, heston(), f, N, n, SEED,
                             mc.Options(path_offset=offset, path_values=True))
    p = mc.mc_price(ctx, heston(), f, N, n, SEED,
                    mc.Options(greeks=3, path_offset=offset, path_values=True))
    assert np.array_equal(p["path_values"][:, 0], a["path_values"][:, 0])
    for c in (1, 2):
        x, y = p["path_values"][:, c], a["path_values"][:, c]
        tol = 4 * n * 2.0 ** -53 * (1.0 + np.abs(y).max())
        assert np.max(np.abs(x - y)) <= tol, c
    assert p["greeks_method"] == mc.MC_GREEKS_PATHWISE


@pytest.mark.parametrize("prec", [mc.MC_FP32, mc.MC_FP64])
@pytest.mark.parametrize("N,n", [(2, 1), (300, 2), (1025, 7)])
def test_heston_payoff_of_its_own_prices_like_rows(ctx, prec, N, n):
    # A price without rows runs its payoff alone: the same paths, so the mean
    # of the rows to FP64 rounding.
    for kind, name in ((mc.MC_EURO_CALL, "euro"), (mc.MC_ASIAN_ARITH_CALL, "asian")):
        f = mc.Payoff(kind, 97.0)
        r = mc.mc_price(ctx, heston(), f, N, n, SEED, mc.Options(prec=prec))
        v = mc.mc_price(ctx, heston(), f, N, n, SEED, mc.Options(prec=prec, path_values=True))
        col = v["path_values"][:, v["path_channels"].index(name)]
        assert abs(r["price"] - col.mean()) <= 1e-13 * N * (1.0 + abs(col.mean()))
        assert r["price"] == v["price"] and r["std_err"] == v["std_err"]


@pytest.mark.parametrize("m_every,N,n,offset", [(1, 130, 3, (1 << 32) - 40), (3, 70, 10, 7),
                                                (5, 65, 5, (1 << 33) - 64), (7, 129, 6, 0),
                                                (2, 300, 9, (1 << 32) - 257)])
def test_learned_cv_segments_and_straddles(ctx, m_every, N, n, offset):
    # Segments that begin on either half of a Philox block, a last segment cut
    # short, waves that straddle a multiple of 2^32; tolerances of the FP32
    # evaluation against the oracle.
    print("cv segments", m_every, N, n, offset, flush=True)
    th = (synth.glorot_mlp() + np.random.default_rng(3).normal(0.0, 0.05, 4545)).astype(np.float32)
    r = mc.mc_price(ctx, heston(), mc.Payoff(mc.MC_ASIAN_ARITH_CALL, H["K"], cv=mc.MC_CV_LEARNED),
                    N, n, SEED, mc.Options(cv_weights=th, cv_hedge_every=m_every, cv_beta=1.0,
                                           path_offset=offset, path_values=True))
    o = oracle.heston_cv(H, n, th.astype(np.float64), N, SEED, path0=offset, m_every=m_every)
    pv = r["path_values"]
    np.testing.assert_allclose(pv[:, 0], o[:, 0], rtol=3e-4, atol=3e-4)
    assert np.abs(pv[:, 1] - o[:, 1]).max() < 2e-3 * (1 + np.abs(o[:, 1]).max())


@pytest.mark.parametrize("payoff,scheme", [
    (mc.MC_EURO_CALL, mc.MC_LOG_EULER), (mc.MC_ASIAN_ARITH_CALL, mc.MC_LOG_EULER),
    (mc.MC_ASIAN_GEO_CALL, mc.MC_LOG_EULER), (mc.MC_UO_BARRIER_CALL, mc.MC_LOG_EULER),
    (mc.MC_UO_BRIDGE_CALL, mc.MC_LOG_EULER), (mc.MC_EURO_CALL, mc.MC_EULER_S),
    (mc.MC_ASIAN_ARITH_CALL, mc.MC_EULER_S), (mc.MC_UO_BARRIER_CALL, mc.MC_EULER_S)])
@pytest.mark.parametrize("N,n,offset", [(2, 1, 0), (257, 3, 2**32 - 100), (70001, 9, 5)])
def test_bumped_paths_in_one_pass(ctx, payoff, scheme, N, n, offset):
    """The finite differences equal the means of explicit bumped FP64 runs,
    for each greek alone and for both, whatever the price run's precision.
    A payoff's last digits may differ between functional sets by a fused
    multiply-add: 4 ulp of a price of 256, over the bump's width."""
    h, S0, sig = 1e-3, 100.0, 0.25
    f = mc.Payoff(payoff, 100.0, B=130.0)

    def model(S=S0, s=sig):
        return mc.Model(kind=mc.MC_GBM, S0=S, r=0.03, T=1.0, sigma=s, scheme=scheme)
    o64 = mc.Options(prec=mc.MC_FP64, path_values=True, path_offset=offset)
    name = {mc.MC_EURO_CALL: "euro", mc.MC_ASIAN_ARITH_CALL: "asian", mc.MC_ASIAN_GEO_CALL: "geo",
            mc.MC_UO_BARRIER_CALL: "uo", mc.MC_UO_BRIDGE_CALL: "uo_bridge"}[payoff]
    col = mc.mc_path_channels(model(), f, o64).index(name)

    def values(m):
        return np.asarray(mc.mc_price(ctx, m, f, N, n, SEED, o64)["path_values"])[:, col]
    want = {"delta": (values(model(S=S0 * (1 + h))) - values(model(S=S0 * (1 - h)))) / (2 * h * S0),
            "vega": (values(model(s=sig * (1 + h))) - values(model(s=sig * (1 - h)))) / (2 * h * sig)}
    width = {"delta": 2 * h * S0, "vega": 2 * h * sig}
    bits = {"delta": mc.MC_GREEK_DELTA, "vega": mc.MC_GREEK_VEGA}
    for wanted in (("delta",), ("vega",), ("delta", "vega")):
        for prec in (mc.MC_FP32, mc.MC_FP64):
            r = mc.mc_price(ctx, model(), f, N, n, SEED, mc.Options(
                prec=prec, path_offset=offset, greeks=sum(bits[g] for g in wanted),
                greeks_method=mc.MC_GREEKS_FD_CRN, fd_rel_step=h))
            for g in wanted:
                tol = 4 * 256 * 2.0**-52 / width[g]
                assert r[g] == pytest.approx(want[g].mean(), rel=1e-12, abs=tol)
                assert r[g + "_se"] == pytest.approx(want[g].std(ddof=1) / math.sqrt(N), rel=1e-9,
                                                     abs=tol)


@pytest.mark.parametrize("d,degree,M,N,n_oos,offset", [
    (1, 1, 1, 300, 0, 0), (2, 2, 3, 1025, 5, (1 << 32) - 500), (4, 1, 2, 70000, 300, 9),
    (3, 2, 4, (1 << 20) + 4097, 0, 1)])
def test_lsm_sweeps_and_reductions(ctx, d, degree, M, N, n_oos, offset):
    """Stages of one and of many rounds of quads, swept in either direction,
    ragged path counts, a straddle of 2^32, no out-of-sample stage: prices
    equal the oracle's up to the FP32 states (2e-6 of the strike over the
    standard error's sqrt(N) paths), counts in the money up to the paths
    within FP32 rounding of the strike."""
    S0, sigma, K = np.full(d, 100.0), 0.2 + 0.03 * np.arange(d), 100.0
    kind = PUT if d == 1 else MAXC
    corr = np.full((d, d), 0.3) + 0.7 * np.eye(d)
    model = mc.Model(kind=mc.MC_GBM if d == 1 else mc.MC_GBM_BASKET, S0=S0, r=0.05, T=1.0,
                     sigma=sigma, corr=corr if d > 1 else None)
    spec = mc.LsmSpec(payoff=kind, K=K, dividend=0.1, n_dates=M, steps_per_date=1, degree=degree,
                      n_paths_oos=n_oos)
    g = mc.mc_price_lsm(ctx, model, spec, N, SEED, mc.Options(path_offset=offset))
    o = oracle.lsm(S0, sigma, np.linalg.cholesky(corr), 0.05, 0.1, 1.0, kind, K, M, 1, degree, N,
                   SEED, path0=offset)
    assert abs(g["price"] - o["price"]) < 2e-6 * K
    n_itm = np.asarray(g["n_itm"], dtype=float)[:M]
    assert np.abs(n_itm - o["n_itm"][:M]).max() <= 1 + 1e-6 * N


@pytest.mark.parametrize("prec", [mc.MC_FP32, mc.MC_BF16_GEMM])
def test_basket_factor_follows_the_matrix(ctx, prec):
    """The factor kept from the last call is used for equal contents only:
    changed in place, of another dimension and back again, each call equals a
    fresh context's, bit for bit."""
    corr = {d: np.full((d, d), 0.3) + 0.7 * np.eye(d) for d in (16, 64)}

    def price(c, d):
        m = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(d, 100.0), r=0.03, T=1.0,
                     sigma=np.linspace(0.1, 0.4, d), corr=corr[d])
        r = mc.mc_price(c, m, mc.Payoff(mc.MC_BASKET_CALL, 100.0), 5000, 3, SEED,
                        mc.Options(prec=prec))
        return r["price"], r["std_err"]

    def fresh(d):
        c = mc.mc_create(0)
        out = price(c, d)
        c.close()
        return out
    for d in (64, 16, 16, 64):
        assert price(ctx, d) == fresh(d)
        corr[d][2, 1] = corr[d][1, 2] = corr[d][1, 2] + 0.1
        assert price(ctx, d) == fresh(d)
    corr[64][0, 1] = 0.2                     # no longer symmetric
    with pytest.raises(Exception, match="symmetric"):
        price(ctx, 64)
    corr[64][0, 1] = corr[64][1, 0]
    assert price(ctx, 64) == fresh(64)


@pytest.mark.parametrize("N,alpha,sigma,mu,strike", [
    (2, 0.5, 0.2, 0.05, 1.0), (513, 0.9, 0.2, 0.05, 1.0), (70001, 0.99, 0.3, 0.05, 1.0),
    ((1 << 19) + 3, 0.95, 0.3, 0.05, 0.9),   # three digits before the list
    (5000, 0.5, 0.2, 0.05, 50.0),            # every value equal: more than the list holds
    (20011, 0.7, 0.4, 0.05, 2.5),            # ties at one value, and others
    (9001, 0.95, 1e-6, 3.0, 0.0)])           # distinct values that share 24 bits
def test_risk_selection(ctx, N, alpha, sigma, mu, strike):
    """Order statistic and tail count exactly, the tail's mean to the rounding
    of its sum (N values: below N 2^-53, in practice sqrt(N) of it)."""
    d = 16
    corr = np.full((d, d), 0.2) + 0.8 * np.eye(d)
    m = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(d, 100.0), r=0.03, T=1.0,
                 sigma=np.full(d, sigma), corr=corr)
    r = mc.mc_risk(ctx, m, [strike], [1.0], alpha, N, 1, SEED, mu=np.full(d, mu),
                   opts=mc.Options(path_values=True))
    x = np.sort(r["pnl"])
    k = int(math.floor(N * (1.0 - alpha))) + 1
    assert r["k"] == k and r["quantile_pnl"] == x[k - 1]
    tail = x[x < x[k - 1]]
    assert r["n_tail"] == tail.size
    if tail.size:
        assert r["cvar"] == pytest.approx(-tail.mean(), rel=1e-12)
    again = mc.mc_risk(ctx, m, [strike], [1.0], alpha, N, 1, SEED, mu=np.full(d, mu))
    assert again["var"] == r["var"] and again["n_tail"] == r["n_tail"]
    assert again["cvar"] == r["cvar"] or not tail.size


@pytest.mark.parametrize("prec", [mc.MC_FP32, mc.MC_FP16_GEMM])
@pytest.mark.parametrize("d,n,N,offset,reps", [
    (16, 1, 2, 0, 1), (16, 1, 4099, 0, 3), (16, 3, 517, 37, 2), (16, 4, 1000, (1 << 32) - 1000, 2),
    (48, 1, 333, 61, 2), (64, 1, 64, 64, 64), (16, 1, 1 << 17, 5, 2)])
def test_qmc_tiles(ctx, prec, d, n, N, offset, reps):
    """Replicates of few dimensions against the run of one replicate that
    writes its per-path values (the general kernel, whose first replicate has
    the same shift): the same values per path, so the means agree to their
    summation, N 2^-53 at worst; and every replicate against the oracle's
    points is covered by the general tests through this route."""
    corr = np.full((d, d), 0.2) + 0.8 * np.eye(d)
    m = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(d, 100.0), r=0.03, T=1.0,
                 sigma=np.linspace(0.1, 0.4, d), corr=corr)
    f = mc.Payoff(mc.MC_BASKET_CALL, 100.0)
    a = mc.mc_price_qmc(ctx, m, f, N, n, SEED, reps, mc.Options(prec=prec, path_offset=offset))
    b = mc.mc_price_qmc(ctx, m, f, N, n, SEED, 1,
                        mc.Options(prec=prec, path_offset=offset, path_values=True))
    assert a["replicate_price"][0] == pytest.approx(b["replicate_price"][0], rel=1e-12, abs=1e-12)
    assert a["replicate_geo"][0] == pytest.approx(b["replicate_geo"][0], rel=1e-12, abs=1e-12)


@pytest.mark.parametrize("wide,narrow,n,m_every", [(32768, 32512, 4, 1), (65536, 65280, 3, 2)])
def test_cv_gradient_of_wide_workgroups(ctx, wide, narrow, n, m_every):
    """Minibatches on either side of the line between workgroups of four and
    of eight waves (1016 and 1024 tiles over two waves; 2040 and 2048 over
    one). The paths they share cancel in the
    difference of their gradients, up to the BF16 rounding of dL/dDelta that
    the moved mean changes (2^-9 of each of N segments, at random: 1e-5 of
    the gradient); the rest is the new paths' part, to BF16's 2e-2. A lost
    or doubled tile would show as 1e-3 or 5e-4."""
    hp = {k: synth.HESTON[k] for k in ("S0", "v0", "kappa", "theta", "xi", "rho", "r", "T", "K")}
    model = mc.Model(kind=mc.MC_HESTON, **{k: v for k, v in hp.items() if k != "K"})
    pay = mc.Payoff(mc.MC_ASIAN_ARITH_CALL, hp["K"], cv=mc.MC_CV_LEARNED)
    th = (synth.glorot_mlp() + np.random.default_rng(5).normal(0.0, 0.2, 4545)).astype(np.float32)
    th = th.astype(np.float64)
    g, o = [], []
    for B in (wide, narrow):
        g.append(mc.mc_cv_loss_grad(ctx, model, pay, n, SEED, 2, 64, B, th, hedge_every=m_every,
                                    prec=mc.MC_BF16_GEMM)[1].astype(np.float64))
        o.append(oracle.cv_loss_grad(hp, n, th, B, SEED, tag=2, path0=64, m_every=m_every)[1])
    err = np.linalg.norm((g[0] - g[1]) - (o[0] - o[1]))
    assert err < 0.05 * np.linalg.norm(o[0] - o[1]) + 1e-4 * np.linalg.norm(o[0])


def test_workspace_contract(ctx):
    """A workspace of mc_workspace_bytes serves every kind of run, also where
    the run's own layout is larger or smaller, and one byte less is refused."""
    import torch
    d = 16
    basket = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(d, 100.0), r=0.03, T=1.0,
                      sigma=np.full(d, 0.2), corr=np.eye(d))
    cases = [(basket, mc.Payoff(mc.MC_BASKET_CALL, 100.0), N, dict(prec=p, path_values=pv))
             for N in (300, 100003) for p in (mc.MC_FP32, mc.MC_BF16_GEMM) for pv in (False, True)]
    cases += [(gbm(), mc.Payoff(mc.MC_UO_BARRIER_CALL, G["K"], B=G["B"]), 5000, dict(prec=mc.MC_FP64)),
              (gbm(), mc.Payoff(mc.MC_EURO_CALL, G["K"]), 5000, dict(prec=mc.MC_FP32)),
              (heston(), mc.Payoff(mc.MC_EURO_CALL, 100.0), 5000, dict(prec=mc.MC_FP32))]
    for m, f, N, kw in cases:
        call = mc._Marshal(m, f, mc.Options(**kw), N)
        if kw.get("path_values"):
            call.want_path_values(N, 3)
        need = _abi.load().mc_workspace_bytes(C.byref(call.cm), C.byref(call.cp), N, 5,
                                              C.byref(call.co))
        buf = torch.empty(need, dtype=torch.uint8, device="cuda:0")
        call.co.workspace = buf.data_ptr()
        res = _abi.McResult()

        def run(size):
            call.co.workspace_bytes = size
            return _abi.load().mc_price(ctx.handle, C.byref(call.cm), C.byref(call.cp), N, 5, SEED,
                                        C.byref(call.co), C.byref(res))
        assert run(need) == mc.MC_OK
        assert res.price == mc.mc_price(ctx, m, f, N, 5, SEED, mc.Options(**kw))["price"]
        assert run(need - 1) == -7           # MC_ERR_WORKSPACE


@pytest.mark.parametrize("d", [32, 112, 256])
@pytest.mark.parametrize("N", [64, 5000, 64 * 224 - 1, 64 * 263 + 5])
def test_split_basket_tiles(ctx, d, N):
    """Runs with split tiles give the same values per path as runs where the
    same paths lie in whole tiles (another path offset and count: 225 tiles
    are not split), bit for bit; the portfolio's against its own pnl."""
    n, corr = 2, np.full((d, d), 0.2) + 0.8 * np.eye(d)
    m = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(d, 100.0), r=0.03, T=1.0,
                 sigma=np.linspace(0.1, 0.4, d), corr=corr)
    f = mc.Payoff(mc.MC_BASKET_CALL, 100.0)
    whole = 64 * 225
    for prec in (mc.MC_FP32, mc.MC_BF16_GEMM):
        a = np.asarray(mc.mc_price(ctx, m, f, N, n, SEED, mc.Options(prec=prec, path_values=True))
                       ["path_values"])
        for first in range(0, N, whole):
            b = np.asarray(mc.mc_price(ctx, m, f, whole, n, SEED, mc.Options(
                prec=prec, path_values=True, path_offset=first))["path_values"])
            k = min(whole, N - first)
            assert np.array_equal(a[first:first + k], b[:k])
    pa = mc.mc_risk(ctx, m, [1.0], [1.0], 0.9, N, n, SEED, opts=mc.Options(path_values=True))["pnl"]
    pb = mc.mc_risk(ctx, m, [1.0], [1.0], 0.9, whole, n, SEED,
                    opts=mc.Options(path_values=True))["pnl"]
    k = min(N, whole)
    assert np.array_equal(pa[:k], pb[:k])


def test_results_past_the_contexts_first_pinned_block():
    # 64 exercise dates return more results than the block of mc_create holds;
    # the context then goes on with a larger one, a second context with its own.
    model = mc.Model(kind=mc.MC_GBM, S0=100.0, r=0.05, T=3.0, sigma=0.2)
    spec = mc.LsmSpec(payoff=PUT, K=100.0, dividend=0.02, n_dates=64, degree=2,
                      n_paths_oos=5001)
    asian = mc.Payoff(mc.MC_ASIAN_ARITH_CALL, K=100.0)
    a, b = mc.mc_create(0), mc.mc_create(0)
    try:
        before = mc.mc_price(a, gbm(), asian, 5001, 13, SEED)
        first = mc.mc_price_lsm(a, model, spec, 20011, SEED)
        after = mc.mc_price(a, gbm(), asian, 5001, 13, SEED)
        again = mc.mc_price_lsm(a, model, spec, 20011, SEED)
        other = mc.mc_price_lsm(b, model, spec, 20011, SEED)
    finally:
        a.close()
        b.close()
    for k in ("price", "std_err"):
        assert before[k] == after[k], k
    for k in ("price", "std_err", "price_oos", "european"):
        assert first[k] == again[k] == other[k], k
    assert np.array_equal(first["beta"], other["beta"], equal_nan=True)
    o = oracle.lsm(np.array([100.0]), np.array([0.2]), np.eye(1), 0.05, 0.02, 3.0, PUT, 100.0, 64,
                   1, 2, 20011, SEED)
    # FP32 states move decisions on the exercise boundary only.
    assert abs(first["price"] - o["price"]) < 0.05 * first["std_err"]


@pytest.mark.parametrize("prec", [mc.MC_FP32, mc.MC_BF16_GEMM])
@pytest.mark.parametrize("d,N", [(16, 200003), (16, 1 << 20), (112, 300007)])
def test_equal_paths_have_no_variance(ctx, prec, d, N):
    """Several tiles per workgroup: paths of one value have a variance of
    exactly 0 (their deviations about any one of them are 0), and a spread far
    below the mean keeps its digits (reference: the values about the first)."""
    def market(sigma):
        return mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(d, 100.0), r=0.03, T=1.0,
                        sigma=np.full(d, sigma), corr=np.eye(d))
    f = mc.Payoff(mc.MC_BASKET_CALL, 90.0)
    r = mc.mc_price(ctx, market(0.0), f, N, 1, SEED, mc.Options(prec=prec, greeks=1))
    assert r["std_err"] == 0.0 and r["delta_se"] == 0.0 and r["n_paths"] == N
    r = mc.mc_risk(ctx, market(0.2), [50.0], [3.0], 0.9, N, 1, SEED, opts=mc.Options(prec=prec))
    assert r["pnl_std_err"] == 0.0 and r["pnl_mean"] == -r["premium"]
    r = mc.mc_price(ctx, market(1e-6), f, N, 1, SEED, mc.Options(prec=prec, path_values=True))
    y = r["path_values"][:, 0]
    se = (y - y[0]).std(ddof=1) / math.sqrt(N)
    assert se > 0.0 and r["std_err"] == pytest.approx(se, rel=1e-9)


@pytest.mark.parametrize("reps,N,n", [(64, 64 * 64 * 13, 1), (64, 64 * 2048, 5)])
def test_equal_points_have_their_value_as_mean(ctx, reps, N, n):
    # Thirteen and 64 tiles per lane, in the tile kernel and the general one.
    m = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(16, 100.0), r=0.03, T=1.0, sigma=np.zeros(16),
                 corr=np.eye(16))
    f = mc.Payoff(mc.MC_BASKET_CALL, 90.0)
    one = mc.mc_price_qmc(ctx, m, f, 64, n, SEED, 1, mc.Options(path_values=True))["path_values"]
    r = mc.mc_price_qmc(ctx, m, f, N, n, SEED, reps)
    assert (one == one[0]).all()
    assert set(r["replicate_price"]) == {one[0, 0]} and set(r["replicate_geo"]) == {one[0, 1]}


@pytest.mark.parametrize("prec", [mc.MC_FP32, mc.MC_FP64])
def test_equal_paths_of_persistent_grids(ctx, prec):
    """Eight paths of one value per thread: the rounding of their sum of
    squares leaves no negative variance. (At most 8 y^2 2^-53 of it per
    thread: a standard error below 1e-11 of the price.)"""
    N = 1 << 24
    flat = mc.Model(kind=mc.MC_GBM, S0=100.0, r=0.03, T=1.0, sigma=0.0)
    still = mc.Model(kind=mc.MC_HESTON, S0=100.0, r=0.03, T=1.0, v0=0.0, kappa=1.0, theta=0.0,
                     xi=0.0, rho=0.0)
    for K in (90.0, 91.7, 93.1):
        for m in (flat, still):
            for kind in (mc.MC_EURO_CALL, mc.MC_ASIAN_ARITH_CALL):
                r = mc.mc_price(ctx, m, mc.Payoff(kind, K), N, 2, SEED, mc.Options(prec=prec))
                assert 0.0 <= r["std_err"] < 1e-11 * r["price"], (m.kind, kind, K)
        r = mc.mc_price(ctx, flat, mc.Payoff(mc.MC_EURO_CALL, K), N, 2, SEED, mc.Options(
            prec=prec, greeks=mc.MC_GREEK_DELTA, greeks_method=mc.MC_GREEKS_FD_CRN))
        # A delta's two payoffs are of the size of the price, their difference
        # of its two-thousandth part.
        assert 0.0 <= r["delta_se"] < 1e-11 * abs(r["delta"]), K


@pytest.mark.parametrize("d", [16, 128])
@pytest.mark.parametrize("S", [101.7, 95.03])
def test_basket_of_one_asset_has_its_price(ctx, d, S):
    """The largest price of the asset table is not rounded to FP32: at sigma =
    r = 0 a basket of that asset alone is worth it to FP64 rounding, and so is
    a portfolio of shares whose other prices are 2^-30, up to what a lane's FP32
    sums lose of those (1e-9 of it)."""
    S0, w = np.full(d, 2.0 ** -30), np.zeros(d)
    S0[0], w[0] = S, 1.0
    m = mc.Model(kind=mc.MC_GBM_BASKET, S0=S0, r=0.0, T=1.0, sigma=np.zeros(d), corr=np.eye(d))
    for K in (0.0, 90.1):
        for prec in (mc.MC_FP32, mc.MC_BF16_GEMM):
            r = mc.mc_price(ctx, m, mc.Payoff(mc.MC_BASKET_CALL, K, weights=w), 64, 1, SEED,
                            mc.Options(prec=prec, greeks=1))
            assert r["price"] == pytest.approx(S - K, rel=1e-12)
            assert r["delta"] == pytest.approx(1.0, rel=1e-12)
    r = mc.mc_risk(ctx, m, [0.0], [1.0], 0.9, 64, 1, SEED)
    assert r["pnl_mean"] + r["premium"] == pytest.approx(S0.sum(), rel=1e-9)


def test_basket_sums_carry_no_common_error(ctx):
    """FP32 log-returns of the geometric basket against L' times the sums of
    the device's own normals, both in 64 bits: the roundings of single paths
    average out (1e-7 of a return over the sqrt of 2^14 paths: 1e-9), what is
    common to all stays as a slope. Allowed: 1.4e-9 of the FP32 constant in
    the normals, 2e-9 of L' in three terms, three times the noise. L' is exact
    in few bits here, so that no rounding of its entries hides an error."""
    d, n, N = 16, 8, 1 << 14
    step = math.sqrt(1.0 / n) / math.log(2.0)
    L = np.arange(3, 3 + d) / 64.0
    S = np.array([mc.mc_normals(ctx, SEED, 0, p, 0, n * d).reshape(n, d).sum(0) for p in range(N)])
    sigma = L / step
    m = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.ones(d), r=0.0, T=1.0, sigma=sigma, corr=np.eye(d))
    got = mc.mc_price(ctx, m, mc.Payoff(mc.MC_BASKET_CALL, 0.0), N, n, SEED,
                      mc.Options(path_values=True))["path_values"][:, 1]
    w = float(np.float32(math.log(2.0) / d))              # the asset table holds it in FP32
    drift = np.float32(-0.5 * sigma * sigma / math.log(2.0)).astype(np.float64)
    want = w * (S @ L)
    slope = ((np.log(got) - w * drift.sum()) * want).sum() / (want * want).sum()
    assert abs(slope - 1.0) < 1.4e-9 + 2e-9 + 3e-9


@pytest.mark.parametrize("d", [64, 128, 256])
def test_basket_sums_over_assets(ctx, d):
    """At sigma = r = 0 a basket is the sum of its FP32 asset table, so what
    is left is the rounding of that sum: fours and a lane's fours in FP32, the
    lanes in FP64. For random weights 1.5e-8 of the sum (root mean square, from
    the FP32 sums in numpy), allowed is twice that; one by one and over the
    lanes in FP32 it is 4.3e-8 to 4.6e-8."""
    rng, err = np.random.default_rng(d), []
    for _ in range(100):
        w = rng.random(d) / d
        m = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(d, 100.0), r=0.0, T=1.0, sigma=np.zeros(d),
                     corr=np.eye(d))
        r = mc.mc_price(ctx, m, mc.Payoff(mc.MC_BASKET_CALL, 0.0, weights=w), 2, 1, SEED)
        ratio = (w * 100.0).max() / float(np.float32((w * 100.0).max()))
        table = (w * 100.0 / ratio).astype(np.float32).astype(np.float64)
        err.append(r["price"] / (table.sum() * ratio) - 1.0)
    assert math.sqrt(np.mean(np.square(err))) < 3e-8


def test_paths_left_out_depend_on_the_channels_computed(ctx):
    """S_T overflows FP32 on some paths: alone, the barrier payoff is 0 there
    and every path counts; with rows, whose average payoff is infinite there,
    those paths are left out."""
    N = 5000
    m = mc.Model(kind=mc.MC_GBM, S0=100.0, r=84.1, T=1.0, sigma=0.25)   # S0 e^84.1 = 3.4e38
    f = mc.Payoff(mc.MC_UO_BARRIER_CALL, 100.0, B=125.0)
    alone = mc.mc_price(ctx, m, f, N, 4, SEED)
    assert (alone["n_paths"], alone["n_nonfinite"], alone["price"]) == (N, 0, 0.0)
    rows = mc.mc_price(ctx, m, f, N, 4, SEED, mc.Options(path_values=True))
    out = ~np.isfinite(rows["path_values"]).all(1)
    assert 0 < out.sum() < N
    assert (rows["n_paths"], rows["n_nonfinite"]) == (N - out.sum(), out.sum())
    assert rows["price"] == 0.0


@pytest.mark.parametrize("d,degree,M,spd,n_oos,offset", [
    (2, 2, 3, 1, 5, 0), (2, 2, 3, 1, 1000, (1 << 32) - 500), (1, 3, 5, 2, 257, (1 << 32) - 3),
    (4, 1, 2, 1, 300, 9), (3, 2, 4, 1, 4099, (1 << 33) - 70)])
def test_lsm_fresh_paths(ctx, d, degree, M, spd, n_oos, offset):
    """Out of sample, the fitted rule on fresh paths, the last waves partial
    and some across a multiple of 2^32: each value the oracle's under the same
    coefficients, except where FP32 states decide otherwise at the exercise
    boundary (at most one path), and their mean the price."""
    S0, sigma, K, N = np.full(d, 100.0), 0.2 + 0.03 * np.arange(d), 100.0, 20011
    kind = PUT if d == 1 else MAXC
    corr = np.full((d, d), 0.3) + 0.7 * np.eye(d)
    model = mc.Model(kind=mc.MC_GBM if d == 1 else mc.MC_GBM_BASKET, S0=S0, r=0.05, T=1.0,
                     sigma=sigma, corr=corr if d > 1 else None)
    spec = mc.LsmSpec(payoff=kind, K=K, dividend=0.1, n_dates=M, steps_per_date=spd, degree=degree,
                      n_paths_oos=n_oos)
    g = mc.mc_price_lsm(ctx, model, spec, N, SEED, mc.Options(path_offset=offset), want_paths=True)
    assert np.asarray(g["beta_valid"])[:M - 1].all()
    nf = g["n_features"]
    o = oracle.lsm_oos(S0, sigma, np.linalg.cholesky(corr), 0.05, 0.1, 1.0, kind, K, M, spd, degree,
                       np.asarray(g["beta"])[:M, :nf], n_oos, SEED, tag=7, path0=offset)
    same = g["oos_exercise_date"] == o["ex"]
    assert (~same).sum() <= 1
    np.testing.assert_allclose(g["oos_value"][same], o["Y"][same], rtol=1e-5, atol=3e-5 * K)
    assert g["price_oos"] == pytest.approx(g["oos_value"].mean(), rel=1e-12)
    assert g["std_err_oos"] == pytest.approx(g["oos_value"].std(ddof=1) / math.sqrt(n_oos), rel=1e-9)


@pytest.mark.parametrize("prec", [mc.MC_BF16_GEMM, mc.MC_FP16_GEMM, mc.MC_BF16X2_GEMM])
@pytest.mark.parametrize("d,N,n", [(16, 130, 1), (32, 67, 2), (96, 67, 1), (256, 65, 2)])
def test_reduced_forms_path_by_path(ctx, prec, d, N, n):
    """Every path but those with a normal on the other side of a rounding
    boundary (one normal in 2^14 within FP32 error of one, counted twice;
    the count's mean plus four of its standard deviations plus one, which is
    below N) has the value of the 64-bit model of its form."""
    sigma, corr, _ = synth.basket_market(d)
    S0, w, K, r_, T = np.full(d, 100.0), np.full(d, 1.0 / d), 40.0, 0.05, 1.0
    r = mc.mc_price(ctx, mc.Model(kind=mc.MC_GBM_BASKET, S0=S0, r=r_, T=T, sigma=sigma, corr=corr),
                    mc.Payoff(mc.MC_BASKET_CALL, K, weights=w), N, n, SEED,
                    mc.Options(prec=prec, path_values=True))
    L = np.linalg.cholesky(corr) * (sigma * np.sqrt(T / n) / np.log(2.0))[:, None]
    Lr = _rounded(L, prec)
    if prec == mc.MC_BF16X2_GEMM:
        Lr = Lr + _bf16(L - Lr)
    x = np.array([Lr @ _rounded(oracle.normals(SEED, 0, p, 0, n * d).reshape(n, d), prec).sum(0)
                  for p in range(N)])
    E = 2.0 ** (x + (r_ - 0.5 * sigma * sigma) * T / np.log(2.0))
    ref = np.exp(-r_ * T) * np.maximum((E * S0 * w).sum(1) - K, 0.0)
    moved = int((np.abs(r["path_values"][:, 0] - ref) > 4e-6 * 100.0).sum())
    mean = N * 2.0 * n * d * 2.0 ** -14
    assert moved <= mean + 4.0 * math.sqrt(mean) + 1.0 < N
