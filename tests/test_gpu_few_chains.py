"""Launches of few long chains: eight waves share 64 paths (or lanes of split
paths), and every sample equals the one that a fixed launch shape, which keeps
a path in one wave, computes."""
import numpy as np
import pytest
import torch

from paper_1505_00965_amd import mlmc as A

pytestmark = pytest.mark.gpu

# kind, scheme, antithetic, payoff, M, level, precision: both models and
# precisions, the twin with and without its own coarse path, rounds of every
# remainder (16, 64, 32 and 256 generator blocks over six or five waves)
CASES = [
    (A.HESTON, 0, 0, A.CALL, 4, 3, 32),
    (A.HESTON, 0, 0, A.LOOKBACK, 2, 7, 64),
    (A.HESTON, 0, 1, A.LOOKBACK, 2, 6, 32),
    (A.HESTON, 0, 0, A.ASIAN, 4, 4, 32),
    (A.GBM, 0, 0, A.LOOKBACK, 4, 3, 64),
    (A.GBM, 1, 1, A.ASIAN, 2, 7, 32),
    (A.GBM, 0, 0, A.DIGITAL_COND, 4, 5, 32),
    (A.GBM, 0, 1, A.DIGITAL_COND, 2, 6, 64),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("N", [1, 64, 1001, 32768])
def test_unsplit_samples_equal_plain_kernel(gctx, case, N):
    kind, scheme, anti, pay, M, l, prec = case
    m, p = A.model(kind, scheme=scheme, antithetic=anti), A.payoff(pay)
    with A.Context(0) as plain:
        plain.set_launch(64, 1)
        out = []
        for c in (gctx, plain):
            d = torch.full((2, N), -1.0, dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()              # the fill runs on another stream
            r = c.mlmc_level_paths(m, p, l, M, N, 3, d[0], d[1], path_offset=77, precision=prec)
            out.append((d.cpu().numpy(), r))
    assert np.array_equal(out[0][0], out[1][0])
    # N summands each, in another order: N eps of their absolute sum
    scale = {k: np.abs(v).sum() for k, v in
             {"sum_y": out[0][0][0] - out[0][0][1], "sum_y2": (out[0][0][0] - out[0][0][1]) ** 2}.items()}
    for k, s in scale.items():
        assert abs(out[0][1][k] - out[1][1][k]) <= 4e-16 * N * s


# 64 lanes a path (32 at 767): one path, the rule's last count with 64 steps a
# lane, and a ragged count beside it
@pytest.mark.parametrize("pay", [A.CALL, A.ASIAN, A.LOOKBACK, A.DIGITAL])
@pytest.mark.parametrize("scheme,M,l,N", [(0, 4, 6, 1), (1, 4, 6, 512), (0, 4, 7, 767), (1, 2, 13, 333)])
def test_split_samples_equal_plain_kernel(gctx, pay, scheme, M, l, N):
    m, p = A.model(A.GBM, scheme=scheme), A.payoff(pay)
    d = torch.full((4, N), -1.0, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()              # the fill runs on another stream
    gctx.mlmc_level_paths(m, p, l, M, N, 5, d[0], d[1], path_offset=9)
    with A.Context(0) as plain:
        plain.set_launch(64, 1)
        plain.mlmc_level_paths(m, p, l, M, N, 5, d[2], d[3], path_offset=9)
    a = d.cpu().numpy()
    assert np.array_equal(a[:2], a[2:])


def test_uncoupled_paths_equal_plain_kernel(gctx):
    """Standard Monte Carlo: no coarse path."""
    with A.Context(0) as plain:
        plain.set_launch(64, 1)
        for m, prec in ((A.model(A.HESTON), 32), (A.model(A.GBM), 32), (A.model(A.GBM), 64)):
            r = [c.mlmc_stdmc(m, A.payoff(A.ASIAN), 4, 4, 300, 11, precision=prec) for c in (gctx, plain)]
            for k in ("sum_y", "sum_y2", "sum_pf", "sum_pc"):
                # 300 positive summands in another order
                assert abs(r[0][k] - r[1][k]) <= 300 * 2.3e-16 * abs(r[1][k])


# sample counts on both sides of a change of the default samples per lane
@pytest.mark.parametrize("kind,l", [(A.GBM, 3), (A.HESTON, 3)])
@pytest.mark.parametrize("N", [262144, 262145, 327680, 327681, 393217, 458753])
def test_sums_do_not_depend_on_samples_per_lane(gctx, kind, l, N):
    m, p = A.model(kind), A.payoff(A.LOOKBACK)
    r = gctx.mlmc_level(m, p, l, 4, N, 21, path_offset=5)
    with A.Context(0) as plain:
        plain.set_launch(256, 2)
        ref = plain.mlmc_level(m, p, l, 4, N, 21, path_offset=5)
    assert r["n"] == ref["n"] == N
    for k, k2 in (("sum_y", "sum_y2"), ("sum_pf", "sum_pf2"), ("sum_pc", "sum_pc2")):
        # N summands in another order, their absolute sum at most sqrt(N sum x^2)
        assert abs(r[k] - ref[k]) <= 2 * N * 2.0 ** -53 * (N * ref[k2]) ** 0.5
        assert abs(r[k2] - ref[k2]) <= 2 * N * 2.0 ** -53 * ref[k2]
