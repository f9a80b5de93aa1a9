"""Published sums: calls that leave the context's records to the next one,
in every order, and the randomised estimator's two forms."""
import numpy as np
import pytest

from paper_1505_00965_amd import mlmc
from paper_1505_00965_amd import workloads as W

pytestmark = pytest.mark.gpu


def same(a, b):
    # the same samples summed in another order: a few ulps of sum |Y|
    s = (a["n"] * a["sum_y2"]) ** 0.5
    assert abs(a["sum_y"] - b["sum_y"]) <= 1e-12 * s + 1e-300
    assert abs(a["sum_y2"] - b["sum_y2"]) <= 1e-12 * a["sum_y2"] + 1e-300
    assert a["n"] == b["n"] and a["n_nonfinite"] == b["n_nonfinite"]


def test_calls_in_turn_leave_zeros(tmp_path):
    gm, gp = mlmc.model(**W.GBM_MODEL), mlmc.payoff(**W.CALL)
    mil = mlmc.model(**dict(W.GBM_MODEL), scheme=1)
    huge = mlmc.model(**dict(W.GBM_MODEL, sigma=1e30))    # every path overflows
    with mlmc.Context(0) as ctx:
        ref = ctx.mlmc_level(gm, gp, 2, 4, 1000, 7)
        refb = ctx.mlmc_levels_batch(gm, [gp, gp], 4, 2, [[500, 40, 7], [3, 0, 9]], 5)
        others = [
            lambda: ctx.mlmc_level(gm, gp, 0, 4, 100003, 3, precision=64),
            lambda: ctx.mlmc_rhee_glynn(mil, gp, 4, 5, 0.125, 20011, 3),
            lambda: ctx.mlmc_rhee_glynn(mil, gp, 2, 3, 0.3, 501, 3, precision=64),
            lambda: ctx.mlmc_stdmc(gm, gp, 3, 2, 4099, 3),
            lambda: ctx.autotune(gm, gp, M=4, precision=32, cache_path=str(tmp_path / "t.json")),
            lambda: ctx.mlmc_run(gm, gp, 0.5, persistent=True),
            lambda: ctx.mlmc_level(huge, gp, 6, 4, 77, 3, allow_nonfinite=True),
            lambda: ctx.set_timing(True), lambda: ctx.mlmc_level(gm, gp, 1, 4, 999, 3),
            lambda: ctx.set_timing(False),
        ]
        for k, f in enumerate(others):
            print("after", k, flush=True)
            f()
            same(ref, ctx.mlmc_level(gm, gp, 2, 4, 1000, 7))
            got = ctx.mlmc_levels_batch(gm, [gp, gp], 4, 2, [[500, 40, 7], [3, 0, 9]], 5)
            for ra, rb in zip(refb, got):
                for a, b in zip(ra, rb):
                    same(a, b)


# L = 0 has no bin edge; q near 1 gives every level a share; N around a wave
@pytest.mark.parametrize("M,L,q,N", [(4, 0, 0.5, 65), (4, 4, 0.125, 100003), (2, 7, 0.9, 5001), (2, 3, 0.4, 1)])
def test_randomised_estimate_by_plan_and_by_level(gctx, M, L, q, N):
    mil, gp = mlmc.model(**dict(W.GBM_MODEL), scheme=1), mlmc.payoff(**W.ASIAN)
    a = gctx.mlmc_rhee_glynn(mil, gp, M, L, q, N, 11)
    gctx.set_timing(True)                 # a launch per level
    b = gctx.mlmc_rhee_glynn(mil, gp, M, L, q, N, 11)
    gctx.set_timing(False)
    assert a["N"] == b["N"] and sum(a["N"]) == N
    # the draws: level l above l - 1 when the uniform is at least F_(l-1)
    import torch
    w = torch.zeros(4 * ((N + 3) // 4), dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()              # the fill runs on another stream than the words
    gctx.mlmc_philox_words(11, 0, 0, 7, 1, (N + 3) // 4, w)
    u = ((w.cpu().numpy().view(np.uint32)[:N] >> 8) + 0.5) * 2.0 ** -24
    F = np.cumsum(a["p"])[:-1]
    assert np.array_equal(np.bincount(np.searchsorted(F, u, side="right"), minlength=L + 1), a["N"])
    for l in range(L + 1):
        s = (a["N"][l] * a["sum_y2"][l]) ** 0.5
        assert abs(a["sum_y"][l] - b["sum_y"][l]) <= 1e-12 * s + 1e-300
        assert abs(a["sum_y2"][l] - b["sum_y2"][l]) <= 1e-12 * a["sum_y2"][l] + 1e-300
