"""What the library's host code does between queueing kernels and reading
their results, on the CPU: libmcpath.so runs on a stand-in for the HIP runtime
(hip_stub.c) in a process of its own."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes as C, sys
sys.path.insert(0, {root!r})
sys.modules["torch"] = None                  # no torch streams or workspaces
stub = C.CDLL({stub!r}, C.RTLD_GLOBAL)
import numpy as np
import paper_1906_02818_amd as mc
from paper_1906_02818_amd import _abi

def cell(name, ctype):
    return ctype.in_dll(stub, name)

d = 16
basket = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(d, 100.0), r=0.03, T=1.0,
                  sigma=np.full(d, 0.2), corr=np.eye(d))
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    from paper_1906_02818_amd import _abi
    if not os.path.exists(_abi.LIB_PATH):
        from paper_1906_02818_amd import build as b
        b.build()
    stub = str(tmp_path_factory.mktemp("stub") / "libhip_stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wall", os.path.join(HERE, "hip_stub.c"),
                    "-o", stub], check=True)

    def go(body):
        code = PRELUDE.format(root=os.path.dirname(HERE), stub=stub) + body
        r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return go


@pytest.mark.parametrize("misses", [0, 1])
def test_risk_waits_for_the_order_statistic(run, misses):
    # With misses = 1 the first finishing pass finds more keys than its list
    # holds; the second one's flag is there before the host looks again, its
    # results are not.
    run(f"""
cell("stub_select_misses", C.c_int).value = {misses}
x = np.array([-12.5])
cell("stub_key", C.c_uint64).value = int(~x.view(np.uint64)[0])
cell("stub_n_tail", C.c_double).value = 7.0
cell("stub_tail_sum", C.c_double).value = -98.0
ctx = mc.mc_create(0)
r = mc.mc_risk(ctx, basket, [1.0], [1.0], 0.9, 1000, 1, 1)
assert (r["quantile_pnl"], r["n_tail"], r["cvar"]) == (-12.5, 7, 14.0), r
""")


def test_noalloc_ignores_the_callers_workspace(run):
    # Whatever workspace the options carry, also one too small for the run.
    run("""
ctx = mc.mc_create(0)
gbm = mc.Model(kind=mc.MC_GBM, S0=100.0, r=0.03, T=1.0, sigma=0.2)
hes = mc.Model(kind=mc.MC_HESTON, S0=100.0, r=0.03, T=1.0, v0=0.04, kappa=2.0, theta=0.04, xi=0.5,
               rho=-0.7)
calls = [(gbm, mc.Payoff(mc.MC_EURO_CALL, 100.0), dict()),
         (gbm, mc.Payoff(mc.MC_UO_BARRIER_CALL, 100.0, B=120.0), dict(prec=mc.MC_FP64)),
         (hes, mc.Payoff(mc.MC_EURO_CALL, 100.0), dict()),
         (hes, mc.Payoff(mc.MC_ASIAN_ARITH_CALL, 100.0), dict(greeks=3))]
for m, f, kw in calls:
    call, res = mc._Marshal(m, f, mc.Options(**kw), 5000), _abi.McResult()
    small = (C.c_char * 16)()
    call.co.workspace, call.co.workspace_bytes = C.addressof(small), 16
    st = _abi.load().mc_price_noalloc(ctx.handle, C.byref(call.cm), C.byref(call.cp), 5000, 8, 1,
                                      C.byref(call.co), C.byref(res))
    assert st == mc.MC_OK, (m, f, kw, mc.mc_last_error(ctx))
""")


def test_basket_rows_stay_in_the_callers_workspace(run):
    # A workspace of the size asked for holds the rows of per-path values,
    # all that grows with the paths; the context adds its factor (8 d^2 bytes)
    # and one block of at most 1 MB. No kernel runs: the rows come back as the
    # workspace held them.
    run("""
for d in (16, 112, 256):
    m = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(d, 100.0), r=0.03, T=1.0, sigma=np.full(d, 0.2),
                 corr=np.eye(d))
    for prec in (mc.MC_FP32, mc.MC_BF16_GEMM, mc.MC_BF16X2_GEMM):
        for N in (3000, 64 * 4096, 1 << 20):         # no split tiles
            f = mc.Payoff(mc.MC_BASKET_CALL, 100.0)
            call, res = mc._Marshal(m, f, mc.Options(prec=prec), N), _abi.McResult()
            call.want_path_values(N, 3)
            need = _abi.load().mc_workspace_bytes(C.byref(call.cm), C.byref(call.cp), N, 100,
                                                  C.byref(call.co))
            for size in (need, need + (1 << 20)):
                ws = np.full(size // 8 + 1, 7.0)
                call.path_buf[:] = 0.0
                call.co.workspace, call.co.workspace_bytes = ws.ctypes.data, size
                ctx = mc.mc_create(0)
                before = cell("stub_malloc_bytes", C.c_uint64).value
                st = _abi.load().mc_price(ctx.handle, C.byref(call.cm), C.byref(call.cp), N, 100, 1,
                                          C.byref(call.co), C.byref(res))
                more = cell("stub_malloc_bytes", C.c_uint64).value - before
                ctx.close()
                assert st == mc.MC_OK
                split = d > 16 and N == 3000
                assert more <= 8 * d * d + (1 << 20) + (47 * d * 256 + 4096 if split else 0), \
                    (d, prec, N, more)
                assert (call.path_buf == 7.0).all(), (d, prec, N)
""")


def test_failed_calls_leave_nothing_queued(run):
    # Kernels read staged inputs from, and write results to, memory of the
    # context that its next call uses again: wherever a call fails, it has
    # waited for what it had queued, and the same call then succeeds.
    run("""
gbm = mc.Model(kind=mc.MC_GBM, S0=100.0, r=0.03, T=1.0, sigma=0.2)
hes = mc.Model(kind=mc.MC_HESTON, S0=100.0, r=0.03, T=1.0, v0=0.04, kappa=2.0, theta=0.04, xi=0.5,
               rho=-0.7)
wide = mc.Model(kind=mc.MC_GBM_BASKET, S0=np.full(256, 100.0), r=0.03, T=1.0,
                sigma=np.full(256, 0.2), corr=np.eye(256))
pay, asian, call = (mc.Payoff(mc.MC_BASKET_CALL, 100.0), mc.Payoff(mc.MC_ASIAN_ARITH_CALL, 100.0),
                    mc.Payoff(mc.MC_EURO_CALL, 100.0))
fd = dict(greeks=3, greeks_method=mc.MC_GREEKS_FD_CRN)
spec = mc.LsmSpec(payoff=mc.MC_LSM_BASKET_PUT, K=100.0, dividend=0.0, n_dates=64, degree=2, n_paths_oos=500)
levels = [mc.Level(4, mc.MC_FP32, 1000), mc.Level(8, mc.MC_FP32, 500)]
O = mc.Options
calls = [
    lambda c: mc.mc_price(c, gbm, mc.Payoff(mc.MC_ASIAN_ARITH_CALL, 100.0, cv=mc.MC_CV_GEO_ASIAN), 1000, 8, 1),
    lambda c: mc.mc_price(c, gbm, asian, 1000, 8, 1, O(path_values=True)),
    lambda c: mc.mc_price(c, gbm, call, 1000, 8, 1, O(**fd)),
    lambda c: mc.mc_price(c, hes, call, 1000, 8, 1, O(**fd)),
    lambda c: mc.mc_price(c, hes, asian, 1000, 300, 1, O(greeks=3)),
    lambda c: mc.mc_price(c, wide, pay, 3000, 8, 1, O(path_values=True)),
    lambda c: mc.mc_price_qmc(c, basket, pay, 1000, 2, 1, 4),
    lambda c: mc.mc_price_qmc(c, wide, pay, 1000, 2, 1, 4),
    lambda c: mc.mc_price_qmc(c, basket, pay, 1000, 2, 1, 1, O(path_values=True)),
    lambda c: mc.mc_risk(c, basket, [1.0], [1.0], 0.9, 1000, 1, 1, opts=O(path_values=True)),
    lambda c: mc.mc_price_lsm(c, gbm, spec, 1000, 1, want_paths=True),
    lambda c: mc.mc_price_mlmc(c, gbm, call, levels, 1),
]
for n, f in enumerate(calls):
    for k in range(1, 1000):
        ctx = mc.mc_create(0)
        cell("stub_pending", C.c_int).value = 0
        cell("stub_select_misses", C.c_int).value = 1
        cell("stub_fail_at", C.c_int).value = k
        try:
            f(ctx)
            done = cell("stub_fail_at", C.c_int).value > 0
            assert done, (n, k, "failure not reported")
        except mc.McError:
            done = False
        assert cell("stub_pending", C.c_int).value == 0, (n, k, mc.mc_last_error(ctx))
        cell("stub_fail_at", C.c_int).value = 0
        f(ctx)
        ctx.close()
        if done:
            break
    assert k > 2
""")


def test_create_needs_no_reported_clock_rate(run):
    # The rate of the device's constant clock serves the kernel times alone.
    run("""
cell("stub_clock_khz", C.c_int).value = 0
ctx = mc.mc_create(0)
r = mc.mc_price(ctx, mc.Model(kind=mc.MC_GBM, S0=100.0, r=0.03, T=1.0, sigma=0.2),
                mc.Payoff(mc.MC_EURO_CALL, 100.0), 1000, 8, 1)
assert r["price"] == 1.0 and r["kernel_ms"] == 0.0
""")
