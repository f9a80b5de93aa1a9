"""fp64 normals against 80-bit arithmetic on the same generator words: the
table intervals of the logarithm and of the angle, and words at the ends."""
import numpy as np
import pytest

from paper_1505_00965_amd import mlmc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,nsteps,level", [(1, 4, 2), (2, 6, 3), (1, 1, 0)])
def test_normals_fp64_to_the_last_places(dim, nsteps, level, gctx):
    import torch
    n, seed = 1 << 18, 20261
    per = dim * nsteps
    q = 4 // per if per < 4 else 1
    nblk = (per + 3) // 4
    w = torch.zeros(n // q * nblk * 4, dtype=torch.int32, device="cuda:0")
    z = torch.zeros(n * per, dtype=torch.float64, device="cuda:0")
    gctx.mlmc_philox_words(seed, level, 0, 0, nblk, n // q, w)
    gctx.mlmc_normals(seed, level, 0, 0, dim, nsteps, n, 64, z)
    u = ((w.cpu().numpy().view(np.uint32).reshape(-1, 2) >> 8).astype(np.longdouble) + 0.5) \
        * np.longdouble(2) ** -24
    # both ends are drawn (131072 words or more: missed with probability e^-13)
    assert u[:, 0].min() < 1e-4 and u[:, 0].max() > 1 - 1e-4
    log = np.where(u[:, 0] > 0.5, np.log1p(u[:, 0] - 1), np.log(u[:, 0]))
    rho = np.sqrt(-2 * log)
    ang = 2 * np.longdouble("3.14159265358979323846264338327950288") * u[:, 1]
    exact = np.stack([rho * np.cos(ang), rho * np.sin(ang)], 1).reshape(-1, 4 * nblk)[:, :max(per, 4)]
    rho = np.repeat(rho, 2).reshape(-1, 4 * nblk)[:, :max(per, 4)]
    got = z.cpu().numpy().reshape(exact.shape)
    # in units of rho 2^-53: logarithm 0.79 ulp (0.8 in the root), root 1, sine
    # and cosine 0.61, product 1
    assert np.all(np.abs(got - exact) <= 4.0 * 2.0 ** -53 * rho)
