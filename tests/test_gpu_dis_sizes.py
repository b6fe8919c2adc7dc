"""Batched DIS screening (Eq. 7) at the edges of its split: passes of 8, 4 and 2
terms per lane and their remainders, ranges of several passes, tiles and runs
of candidates with one more or one less, every key width, with and without
factors that are exactly zero, and the range and tile knobs."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


def candidates(nq, k, seed):
    """k keys of 1 .. 12 random Paulis on random qubits."""
    rng = np.random.default_rng(seed)
    W = (nq + 63) // 64
    x, z = np.zeros((k, W), np.uint64), np.zeros((k, W), np.uint64)
    for a in range(k):
        for q in rng.choice(nq, size=min(nq, int(rng.integers(1, 13))), replace=False):
            p, b = int(rng.integers(1, 4)), np.uint64(1) << np.uint64(q % 64)
            if p & 1:
                x[a, q // 64] |= b
            if p & 2:
                z[a, q // 64] |= b
    return x, z


@pytest.mark.parametrize("nq,n,n_cand,zeros,knobs", [
    (40, 1, 1, False, {}), (40, 512, 15, False, {}), (64, 513, 17, True, {}), (24, 1024, 256, False, {}),
    (33, 1025, 257, True, {}), (124, 2048, 3, False, {}), (128, 2049, 65, True, {}), (65, 9001, 255, False, {}),
    (100, 30_000, 16, False, {"dis_bucket_ranges": 1}), (100, 5000, 100, True, {"dis_bucket_ranges": 7, "dis_tile": 9}),
    (150, 3000, 33, False, {}), (192, 2500, 40, True, {}), (200, 600, 300, False, {}), (256, 2300, 19, True, {})])
def test_dis_sizes(nq, n, n_cand, zeros, knobs):
    ctx = iqcc.Context(0)
    x, z, c = random_terms(nq, n, 3 * nq + n)
    cx, cz = candidates(nq, n_cand, nq + n_cand)
    th, ph = I.qmf_angles(nq, np.random.default_rng(nq))
    if zeros:
        th[::3] = 0.0
        ph[1::5] = 0.0
    for k, v in knobs.items():
        iqcc.iqcc_set_param(ctx.handle, k, v)
    s = iqcc.Store(ctx, nq, max(n, 16)).load_numpy(x, z, c)
    describe(0, "dis sizes", nq=nq, n=n, n_cand=n_cand, zeros=zeros, knobs=knobs)
    g = iqcc.iqcc_dis_gradients(ctx.handle, s.handle, torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda(),
                                iqcc.to_device_words(cx), iqcc.to_device_words(cz)).cpu().numpy()
    ref = O.dis_gradients(nq, x, z, c, th, ph, cx, cz)
    # rounding: products of nq factors and 12 ratios (each a division) within a
    # few ulp of a value of at most |c|, sums of depth below 128
    tol = (4 * nq + 256) * 2.0 ** -53 * float(np.abs(c).sum())
    assert np.abs(g - ref).max() <= tol, (nq, n, n_cand, np.abs(g - ref).max(), tol)
    s.close(); ctx.close()
