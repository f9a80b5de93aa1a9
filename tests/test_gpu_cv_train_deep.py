"""Control-variate training on deep levels: the points of a batch of ordinary
size are worked off at the rate of a shallower one's.

A step costs its points (fine steps 1.. and coarse steps 1.. of every sample)
and one chain of the deepest level's steps, which the longer batch hides: it
has sixteen times the points and a chain of at most 0.5 ms a launch.  Worked
off in chunks of few samples, each with its chain twice, it took 1.7 times as
long a point."""
import time

import pytest

from paper_1505_00965_amd import mlmc
from paper_1505_00965_amd import workloads as W

pytestmark = pytest.mark.gpu


def points(M, lmax, B):
    return B * sum(M ** l - 1 + (M ** (l - 1) - 1 if l else 0) for l in range(lmax + 1))


@pytest.mark.parametrize("md,d", [(W.GBM_MODEL, 2), (W.HESTON_MODEL, 3)])
def test_deep_batch_keeps_the_rate(gctx, md, d):
    B, M = 16384, 4
    gm, gp = mlmc.model(**md), mlmc.payoff(**W.ASIAN)
    rate = {}
    for lmax in (4, 6):
        cv = mlmc.ControlVariate(gctx, d)
        ms = []
        for _ in range(5):
            t = time.perf_counter()
            cv.train(gm, gp, M, lmax, 1, B)
            ms.append((time.perf_counter() - t) * 1e3)
        cv.close()
        rate[lmax] = min(ms) / points(M, lmax, B)
        print(f"lmax={lmax}: {min(ms):.3f} ms a step", flush=True)
    assert rate[6] <= 1.25 * rate[4]

