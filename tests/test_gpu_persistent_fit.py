"""The all-levels sampler where fewer of its blocks fit the device than its
grid has: small plans use the blocks that are resident at once and the rest
leave, larger ones use all; either way every sample is drawn once."""
import numpy as np
import pytest

from paper_1505_00965_amd import mlmc as A
from paper_1505_00965_amd import workloads as W

pytestmark = pytest.mark.gpu
P = {k: A.payoff(**v) for k, v in W.PAYOFFS.items()}


def tabulated(ctx, d):
    cv = A.ControlVariate(ctx, d)
    cv.set_params(np.random.default_rng(3).uniform(-0.2, 0.2, cv.nparams).astype(np.float32))
    cv.set_tabulated(True)
    return cv


# blocks of 256 a compute unit holds: four by the 32 KB of LDS of the table's
# rows or by registers (M = 2 and several payoffs: 108 and more a lane; 96 fit
# five times), five of the call's at M = 4
@pytest.mark.parametrize("md,M,pays,tab,fit", [
    (W.GBM_MODEL, 4, ["call"], False, 5), (W.GBM_MODEL, 2, ["lookback"], False, 4),
    (W.GBM_MODEL, 2, ["call", "asian", "lookback", "digital"], False, 4), (W.HESTON_MODEL, 4, ["call"], False, 5),
    (W.GBM_MODEL, 4, ["call"], True, 4), (W.HESTON_MODEL, 4, ["call"], True, 4)])
def test_blocks_that_work_fit_the_device(gctx, md, M, pays, tab, fit):
    import torch
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    cv = tabulated(gctx, 3 if md["kind"] else 2) if tab else None
    s = gctx.persistent_shape(A.model(**md), [P[k] for k in pays], M, 8, cv)
    assert s["resident"] == fit and s["grid"] == 5 * cu and s["block"] == 256 and s["ppt"] == 1, s
    if cv:
        cv.close()
    with A.Context(0) as fixed:                 # a shape that was set is used as it is
        fixed.set_persistent_launch(256, 1, 8)
        s = fixed.persistent_shape(A.model(**md), [P[k] for k in pays], M, 8)
        assert s["resident"] == 8 and s["grid"] == 8 * cu


def same(a, b):
    assert a["n"] == b["n"] and a["n_nonfinite"] == b["n_nonfinite"]
    for k in ("sum_y", "sum_pf", "sum_pc"):     # other association: N eps of the absolute sum
        assert abs(a[k] - b[k]) <= 1e-12 * (b["n"] * b[k + "2"]) ** 0.5 + 1e-300, k
        assert abs(a[k + "2"] - b[k + "2"]) <= 1e-12 * b[k + "2"] + 1e-300, k


# plans of no item, of one, of fewer items than resident blocks, between those
# and the grid, of a few per block, and past the rule's end (32768 path steps a
# block of the grid: 42e6) on either side; items of 65536 steps (from 336e6 on)
# and sixteen a block (from 1.34e9 on)
@pytest.mark.parametrize("md", [W.GBM_MODEL, W.HESTON_MODEL])
@pytest.mark.parametrize("N", [[0, 0, 0, 0], [1, 0, 0, 0], [70000, 5000, 700, 90], [3000000, 400000, 30000, 2000],
                               [9000000, 1300000, 300000, 60000], [20000000, 1900000, 400000, 50000],
                               [21000000, 2100000, 500000, 60000], [130000000, 2, 0, 1],
                               [400000000, 1000, 0, 3], [1500000000, 70000, 999, 0]])
def test_every_sample_once(gctx, md, N):
    m, M, L = A.model(**md), 4, 3
    for pays in ([P["lookback"]], [P["lookback"], P["call"]]):
        got = gctx.mlmc_levels_batch(m, pays, M, L, [N] * len(pays), 11)
        with A.Context(0) as fixed:
            fixed.set_persistent_launch(256, 1, 4)
            ref = fixed.mlmc_levels_batch(m, pays, M, L, [N] * len(pays), 11)
        for rg, rr in zip(got, ref):
            for a, b in zip(rg, rr):
                same(a, b)


@pytest.mark.parametrize("md,M", [(W.GBM_MODEL, 4), (W.GBM_MODEL, 2), (W.HESTON_MODEL, 4)])
@pytest.mark.parametrize("eps", [0.2, 0.02, 0.006])
def test_tabulated_runs(gctx, md, M, eps):
    def run(ctx, cv):
        return ctx.mlmc_run(A.model(**md), P["asian"], eps, M=M, L_max=7, n_pilot=3000, seed=5, persistent=True,
                            cv=cv, allow_notconv=True)
    cv = tabulated(gctx, 3 if md["kind"] else 2)
    a = run(gctx, cv)
    cv.close()
    with A.Context(0) as fixed:
        fixed.set_persistent_launch(256, 1, 3)
        cv = tabulated(fixed, 3 if md["kind"] else 2)
        b = run(fixed, cv)
        cv.close()
    assert a["N"] == b["N"] and a["iterations"] == b["iterations"]
    assert np.allclose(a["sum_y2"], b["sum_y2"], rtol=1e-12)
