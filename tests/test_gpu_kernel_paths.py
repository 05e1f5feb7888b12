"""GPU tests of the kernels' branches at the sizes where they can go wrong:
remainders of a Philox block, path indices that straddle 2^32, functional sets
of their own, the edges of tiles. Each is held to the FP64 oracle or to the
general path."""
import numpy as np
import pytest

import oracle
import paper_1906_02818_amd as mc
import synth

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
