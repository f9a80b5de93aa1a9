"""Which launch a level takes: the kernel of few long chains at the counts that
its tests run, on either side of its thresholds, and never under a fixed
shape; the samples per lane at the counts where the default changes."""
import pytest
import torch

from paper_1505_00965_amd import mlmc as A
from test_gpu_few_chains import CASES

pytestmark = pytest.mark.gpu


def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("case", CASES)
def test_few_chains_kernel_is_the_one_compared(gctx, case):
    kind, scheme, anti, pay, M, l, prec = case
    m, p = A.model(kind, scheme=scheme, antithetic=anti), A.payoff(pay)
    for N in (1, 64, 1001, 32768):
        s = gctx.level_shape(m, p, l, M, N, prec)
        assert s["few_chains"] == 1 and s["split"] == 1, (N, s)
    with A.Context(0) as plain:
        plain.set_launch(64, 1)
        assert plain.level_shape(m, p, l, M, 1001, prec)["few_chains"] == 0


@pytest.mark.parametrize("scheme,M,l,N,split", [(0, 4, 6, 1, 64), (1, 4, 6, 512, 64), (0, 4, 7, 767, 64),
                                                (1, 2, 13, 333, 64)])
def test_few_split_chains(gctx, scheme, M, l, N, split):
    m = A.model(A.GBM, scheme=scheme)
    for pay in (A.CALL, A.ASIAN, A.LOOKBACK, A.DIGITAL):
        s = gctx.level_shape(m, A.payoff(pay), l, M, N)
        assert s["few_chains"] == 1 and s["split"] == split, s
    with A.Context(0) as plain:
        plain.set_launch(64, 1)
        s = plain.level_shape(m, A.payoff(A.CALL), l, M, N)
        assert s["few_chains"] == 0 and s["split"] == split     # the split is a choice of N alone


# blocks of 64 chains per compute unit up to which the kernel is taken; none
# below 64 steps, nor for fp32 GBM paths that could be split and are not
@pytest.mark.parametrize("kind,anti,pay,l,prec,per_cu", [
    (A.HESTON, 0, A.CALL, 2, 32, 0), (A.HESTON, 0, A.CALL, 3, 32, 2), (A.HESTON, 1, A.LOOKBACK, 3, 32, 2),
    (A.HESTON, 0, A.CALL, 4, 32, 3), (A.GBM, 0, A.CALL, 4, 64, 3), (A.GBM, 0, A.DIGITAL_COND, 5, 32, 3),
    (A.HESTON, 0, A.LOOKBACK, 4, 64, 3)])
def test_thresholds_of_few_chains(gctx, kind, anti, pay, l, prec, per_cu):
    m, p = A.model(kind, antithetic=anti), A.payoff(pay)
    edge = 64 * cus() * per_cu
    if edge:
        assert gctx.level_shape(m, p, l, 4, edge, prec)["few_chains"] == 1
    s = gctx.level_shape(m, p, l, 4, edge + 1, prec)
    assert s["few_chains"] == 0


# as many blocks a compute unit as can be resident in two rounds: by its
# registers one block of the fp64 conditional digital fits, but for Milstein's
# without the twin; every other variant holds two at least
@pytest.mark.parametrize("kind,scheme,anti", [(A.GBM, 0, 0), (A.GBM, 0, 1), (A.GBM, 1, 0), (A.GBM, 1, 1),
                                              (A.HESTON, 0, 0), (A.HESTON, 0, 1)])
@pytest.mark.parametrize("pay", [A.CALL, A.ASIAN, A.LOOKBACK, A.DIGITAL, A.DIGITAL_COND])
@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("M,l,most", [(4, 3, 2), (4, 4, 3), (2, 10, 3)])
def test_few_chains_within_two_rounds(gctx, kind, scheme, anti, pay, prec, M, l, most):
    m, p, cu = A.model(kind, scheme=scheme, antithetic=anti), A.payoff(pay), cus()
    for blocks in (1, 2, 3):
        N = 64 * cu * blocks
        s = gctx.level_shape(m, p, l, M, N, prec)
        if s["split"] > 1 or prec == 32 and kind == A.GBM and not anti and pay != A.DIGITAL_COND:
            continue                            # decided by the split paths' lanes
        assert s["resident"] >= 1
        if s["few_chains"]:
            assert blocks <= min(most, 2 * s["resident"]), (blocks, s)
            # capped at the blocks that fit, as the rule knows without asking
            assert s["grid"] == cu * min(blocks, s["resident"]), (blocks, s)
        else:
            assert blocks > 2, (blocks, s)


@pytest.mark.parametrize("kind", [A.GBM, A.HESTON])
def test_samples_per_lane(gctx, kind):
    # 256 threads with two samples a lane: 512 samples a block
    m, p, cu = A.model(kind), A.payoff(A.LOOKBACK), cus()
    for N, ppt in ((1024 * cu, 2), (1024 * cu + 1, 1), (1280 * cu, 1), (1280 * cu + 1, 2), (1536 * cu + 1, 1),
                   (1792 * cu + 1, 2)):
        s = gctx.level_shape(m, p, 3, 4, N)
        assert (s["block"], s["ppt"], s["few_chains"]) == (256, ppt, 0), (N, s)
    with A.Context(0) as plain:
        plain.set_launch(256, 2)
        assert plain.level_shape(m, p, 3, 4, 1024 * cu + 1)["ppt"] == 2
