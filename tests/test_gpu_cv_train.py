"""Training kernels of the control variate at their edges: batches that do not
fill a wave or a block, one-step levels only, two-step levels (M = 2), and a
batch whose points exceed the scratch and is worked off in chunks."""
import math

import numpy as np
import pytest

from paper_1505_00965_amd import mlmc
from paper_1505_00965_amd import workloads as W

pytestmark = pytest.mark.gpu
S0 = 100.0


def net(d, seed):
    r = np.random.default_rng(seed)
    n = 64 * d + 64 + 4096 + 64 + 64 + 1
    return (r.uniform(-1, 1, n) * np.sqrt(6.0 / 128)).astype(np.float32)


# B around a wave (64) and a block of samples (256); lmax = 0 has no points
# past t = 0; M = 2 has levels of one and two generator-sharing steps
@pytest.mark.parametrize("kind,pname,M,lmax,B", [
    (0, "call", 4, 0, 65), (0, "asian", 4, 1, 2), (0, "lookback", 2, 3, 63), (0, "digital", 2, 1, 257),
    (1, "call", 4, 2, 321), (1, "asian", 2, 2, 64)])
def test_loss_and_gradient_at_the_edges(gctx, orc, kind, pname, M, lmax, B):
    print(f"case {kind} {pname} M={M} lmax={lmax} B={B}", flush=True)
    md = W.GBM_MODEL if kind == 0 else W.HESTON_MODEL
    gm, om = mlmc.model(**md), orc.model(**md)
    # the digital pays 100: its level differences are of the others' size
    pd = dict(W.PAYOFFS[pname], payout=100.0)
    gp, op = mlmc.payoff(**pd), orc.payoff(**pd)
    d = 3 if kind else 2
    params = net(d, 7)
    cv = mlmc.ControlVariate(gctx, d)
    cv.set_params(params)
    loss, g, var = cv.loss_grad(gm, gp, M, lmax, B, seed=17, step=5)
    emu = orc.CVNet(params.astype(np.float64), d, 64, bf16_emulate=True)
    oloss, og, ovar = orc.cv_loss_grad(om, op, M, lmax, B, 17, 5, emu, nthreads=8)
    cv.close()
    # |dP| <= 1e-4 S0 per payoff, so a sample's Y moves by at most 2e-4 S0 and
    # the batch deviation by sqrt(2) times that (B = 2, the worst n/(n-1))
    bar = math.sqrt(2.0) * 2e-4 * S0
    std, ostd = np.sqrt(var), np.sqrt(np.array(ovar))
    assert np.all(np.abs(std - ostd) <= bar), (std, ostd)
    C = np.array([1.0] + [M ** l + M ** (l - 1) for l in range(1, lmax + 1)])
    assert abs(loss - oloss) <= bar * np.sqrt(C).sum()
    assert abs(loss - (np.sqrt(C) * std).sum()) <= 1e-12 * loss
    assert np.all(np.isfinite(g))
    if B > 2:
        og = np.asarray(og)
        rel = np.linalg.norm(g - og) / np.linalg.norm(og)
        cos = g @ og / (np.linalg.norm(g) * np.linalg.norm(og))
        print(f"gradient rel L2 {rel:.3e} cosine {cos:.8f}")
        assert rel <= 2e-2 and cos >= 0.999


def test_batch_in_chunks(gctx):
    """177 points a sample at M = 2, lmax = 6: 100003 samples exceed 2^24
    points.  Against the same paths and network in fp64 torch (autograd)."""
    import torch
    from perf import cases
    B, M, lmax, seed, step = 100003, 2, 6, 23, 2
    params = net(2, 9)
    cv = mlmc.ControlVariate(gctx, 2)
    cv.set_params(params)
    loss, g, var = cv.loss_grad(mlmc.model(**W.GBM_MODEL), mlmc.payoff(**W.ASIAN), M, lmax, B, seed, step)
    cv.close()
    m = dict(W.GBM_MODEL, scheme=0, antithetic=0)
    q = torch.tensor(params, dtype=torch.float64, device="cuda:0", requires_grad=True)
    phi = cases._phi_of(m, q, "net")
    og = torch.zeros_like(q)
    for l in range(lmax + 1):
        y = torch.cat([f - c for f, c in cases._samples(m, W.ASIAN, M, l, step * B, B, seed, cases.S_TRAIN,
                                                        phi=phi, most=2 ** 40)])
        v = y.var()
        std = math.sqrt(v.item())
        # layer 2 runs in bf16: 2^-9 a product, under 1% of a deviation
        assert abs(math.sqrt(var[l]) - std) <= 1e-2 * std, l
        og += torch.autograd.grad(torch.sqrt(cases._cost(M, l) * v), q)[0]
        del y, v
    torch.cuda.empty_cache()
    og = og.cpu().numpy()
    rel = np.linalg.norm(g - og) / np.linalg.norm(og)
    print(f"gradient rel L2 {rel:.3e}")
    assert rel <= 3e-2
