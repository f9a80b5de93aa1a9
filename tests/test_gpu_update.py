"""The adaptive update on few and on many levels: sums of every level
absorbed, and the fitted rates of the finished run."""
import numpy as np
import pytest

from paper_1505_00965_amd import mlmc as A

pytestmark = pytest.mark.gpu


# deepest level below, at and above 8 (the update's waves take levels w and
# w + 8), one fitted level included (no rate then)
@pytest.mark.parametrize("L", [1, 2, 7, 8, 11])
@pytest.mark.parametrize("persistent", [False, True])
def test_update_absorbs_every_level_and_fits_rates(gctx, L, persistent):
    m, p = A.model(), A.payoff(A.ASIAN)
    r = gctx.mlmc_run(m, p, 5.0, M=2, L_min=L, L_max=L, n_pilot=500, seed=3, persistent=persistent,
                      allow_notconv=True)
    n, s1, s2 = (np.array(r[k][:L + 1]) for k in ("N", "sum_y", "sum_y2"))
    for l in range(L + 1):
        ref = gctx.mlmc_level(m, p, l, 2, int(n[l]), 3)
        # sums of fp32 samples in another order: n summands, 2^-53 each, and
        # their absolute sum at most sqrt(n sum y^2)
        tol = 2 * n[l] * 2.0 ** -53 * np.sqrt(n[l] * ref["sum_y2"])
        assert abs(s1[l] - ref["sum_y"]) <= tol
        assert abs(s2[l] - ref["sum_y2"]) <= 2 * n[l] * 2.0 ** -53 * ref["sum_y2"]
    est, x = s1 / n, np.arange(1, L + 1)
    v = s2 / n - est ** 2
    cost = np.array([2.0 ** l + 2.0 ** (l - 1) for l in x])
    for key, y, sign in (("alpha", np.abs(est[1:]), -1), ("beta", v[1:], -1), ("gamma", cost, 1)):
        if L < 2:
            assert np.isnan(r[key])
        else:
            # a fit of a dozen logarithms in fp64: 1e-12 is 4000 roundings
            assert abs(r[key] - sign * np.polyfit(x, np.log2(y), 1)[0]) <= 1e-12 * 20
