"""The all-levels samplers (M = 4, any payoff but lookback, no control variate)
that take their whole grid as blocks that work, without a look at the plan's
number: all of it fits the device."""
import pytest

from paper_1505_00965_amd import mlmc as A
from paper_1505_00965_amd import workloads as W

pytestmark = pytest.mark.gpu
P = dict({k: A.payoff(**v) for k, v in W.PAYOFFS.items()}, cond=A.payoff(A.DIGITAL_COND))


@pytest.mark.parametrize("pay", [k for k in sorted(P) if k != "lookback"])
@pytest.mark.parametrize("md", [W.GBM_MODEL, dict(W.GBM_MODEL, scheme=1), W.HESTON_MODEL],
                         ids=["gbm", "milstein", "heston"])
def test_five_blocks_fit(gctx, md, pay):
    s = gctx.persistent_shape(A.model(**md), [P[pay]], 4, 6)
    assert s["resident"] == 5, s
