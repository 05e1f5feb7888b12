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
