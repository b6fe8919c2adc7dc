"""Angle gradients (derivative of Eq. 3) at the edges of the split -- no row,
one row, one wave's, one team's and one workgroup's rows and one more, several
workgroups -- for every key width, with coefficients over many decades up to
the fixed-point bound, factors on both sides of the null threshold, and rows in
two orders (the same bits)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,n,special", [
    (20, 0, ""), (20, 1, ""), (31, 64, ""), (32, 65, "tiny"), (33, 256, ""), (64, 257, "wide"), (40, 768, ""),
    (40, 769, "tiny"), (50, 70_001, "wide"), (65, 255, ""), (124, 769, "wide"), (128, 50_000, ""), (100, 3000, "tiny"),
    (150, 385, ""), (192, 20_000, "wide"), (200, 513, "tiny"), (256, 5000, "")])
def test_angle_gradient_sizes(nq, n, special):
    ctx = iqcc.Context(0)
    x, z, c = random_terms(nq, n, 5 * nq + n)
    n = len(c)
    rng = np.random.default_rng(nq + n)
    th, ph = I.qmf_angles(nq, rng)
    if special == "wide":     # up to the bound of the exact sums
        c = c * 2.0 ** rng.uniform(-60, 28, n)
    if special == "tiny":     # sin(theta) about 2^-99.6, 2^-102.9 (null), 2^-53 and 0
        th[1::7], th[2::7], th[3::7], th[4::7] = 1e-30, 1e-31, np.pi, 0.0
    tht, pht = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    rows = []
    for order in (np.arange(n), rng.permutation(n)):
        s = iqcc.Store(ctx, nq, max(n, 16)).load_numpy(x[order], z[order], c[order])
        describe(0, "angle gradient sizes", nq=nq, n=n, special=special)
        lam = torch.zeros(iqcc.iqcc_store_rows(s.handle), dtype=torch.float64, device="cuda")
        dt, dp = iqcc.iqcc_qmf_energy_backward(ctx.handle, s.handle, tht, pht, None, lam)
        rows.append((dt.cpu().numpy(), dp.cpu().numpy()))
        sx, sz, _ = s.to_numpy()
        ref = O.expectations(nq, sx, sz, th, ph) if n else np.zeros(0)
        got = lam[:n].cpu().numpy()       # a loaded store holds its terms in the first rows, in export order
        assert np.abs(got - ref).max(initial=0.0) <= 4 * nq * 2.0 ** -53
        s.close()
    assert np.array_equal(rows[0][0], rows[1][0]) and np.array_equal(rows[0][1], rows[1][1])
    rt, rp = O.qmf_grad_angles(nq, x, z, c, th, ph) if n else (np.zeros(nq), np.zeros(nq))
    # products of nq factors and a division within a few ulp of values of at
    # most |c|, three sigmas, and the left-out contributions below 2^-69 |c|
    tol = 3 * (4 * nq + 64) * 2.0 ** -53 * float(np.abs(c).sum()) + 1e-300
    assert np.abs(rows[0][0] - rt).max() <= tol and np.abs(rows[0][1] - rp).max() <= tol, (nq, n, special)
    ctx.close()
