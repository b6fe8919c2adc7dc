"""Batched DIS screening on both sides of the counts of terms and candidates at
which the term ranges are halved, once and twice."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import describe
from tests.test_gpu_dis_sizes import candidates
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,n,n_cand", [(40, 130_000, 1), (40, 262_000, 1), (40, 270_000, 2), (100, 33_000, 112),
                                         (100, 33_000, 130), (150, 20_000, 17), (70, 3000, 33)])
def test_dis_ranges(nq, n, n_cand):
    describe(nq, "dis ranges", n=n, n_cand=n_cand)
    ctx = iqcc.Context(0)
    x, z, c = random_terms(nq, n, nq + n)
    cx, cz = candidates(nq, n_cand, nq + n_cand)
    th, ph = I.qmf_angles(nq, np.random.default_rng(nq))
    s = iqcc.Store(ctx, nq, len(c)).load_numpy(x, z, c)
    g = iqcc.iqcc_dis_gradients(ctx.handle, s.handle, torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda(),
                                iqcc.to_device_words(cx), iqcc.to_device_words(cz)).cpu().numpy()
    pick = np.unique(np.linspace(0, n_cand - 1, 6).astype(int))   # (the oracle is serial)
    ref = O.dis_gradients(nq, x, z, c, th, ph, cx[pick], cz[pick])
    # as for the sizes: nq factors and 12 ratios per term, sums of depth below 128
    tol = (4 * nq + 256) * 2.0 ** -53 * float(np.abs(c).sum())
    assert np.abs(g[pick] - ref).max() <= tol
    s.close(); ctx.close()
