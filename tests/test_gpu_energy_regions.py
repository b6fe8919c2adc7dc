"""Stand-alone energy of stores in bucket regions, whose workgroups differ for
two-word keys: one term, a workgroup's rows and one more, more groups of
buckets than one workgroup takes."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import describe
from tests.test_gpu_energy_sizes import random_terms
from tests.test_gpu_inplace import INPLACE, _Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [40, 65, 128, 150])
@pytest.mark.parametrize("n,per_bucket", [(1, 256), (1024, 256), (1025, 8), (4097, 1000), (70_001, 16)])
def test_energy_regions(nq, n, per_bucket):
    describe(nq, "energy regions", n=n, per_bucket=per_bucket)
    ctx = iqcc.Context(0)
    x, z, c = random_terms(nq, n, nq + n)
    th, ph = I.qmf_angles(nq, np.random.default_rng(nq))
    tht, pht = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    with _Params(ctx, inplace_bucket_terms=per_bucket):
        s = iqcc.Store(ctx, nq, max(2 * len(c), 64), INPLACE).load_numpy(x, z, c)
    got = [float(iqcc.iqcc_qmf_energy(ctx.handle, s.handle, tht, pht).item()) for _ in range(2)]
    # as for loaded rows: nq multiplications per term, sums of depth below 128
    tol = (4 * nq + 128) * 2.0 ** -53 * float(np.abs(c).sum())
    assert got[0] == got[1]
    assert abs(got[0] - O.qmf_energy(nq, x, z, c, th, ph)) <= tol
    s.close(); ctx.close()
