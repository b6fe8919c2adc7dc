"""In-place steps whose items hold one pair of buckets (row positions from
ballots) and many (from the general ranks), with more and with fewer freed rows
than new keys, stashes of one and of several slices, and relocated items."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms
from tests.test_gpu_inplace import INPLACE, _Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,n", [(30, 3000), (124, 3000), (200, 1500)])
@pytest.mark.parametrize("per_bucket", [8, 64, 150, 1000])
@pytest.mark.parametrize("eps", [1e-3, 0.4])
def test_inplace_slots(nq, n, per_bucket, eps):
    ctx = iqcc.Context(0)
    x, z, c = random_terms(nq, n, nq + per_bucket)
    rng = np.random.default_rng(nq)
    th, ph = I.qmf_angles(nq, rng)
    tht, pht = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    ents = [I.single_qubit_pauli(nq, p) for p in ("XYZ", "IZXXY", "XYZ")]
    e = torch.zeros(3, dtype=torch.float64, device="cuda")
    with _Params(ctx, inplace_bucket_terms=per_bucket):
        s = iqcc.Store(ctx, nq, 8 * n, INPLACE).load_numpy(x, z, c)
    for j, (px, pz) in enumerate(ents):
        describe(j, "inplace slots", nq=nq, n=n, per_bucket=per_bucket, eps=eps)
        iqcc.iqcc_dress_inplace(ctx.handle, s.handle, px, pz, 0.5 + 0.2 * j, eps, tht, pht,
                                e[j - 1:j] if j else None, e[j:j + 1])
        x, z, c = O.dress(nq, x, z, c, px, pz, 0.5 + 0.2 * j, eps)
        assert_same_terms(s.to_numpy(), (x, z, c), f"step {j}")
        assert s.count() == len(c)
        ref = O.qmf_energy(nq, x, z, c, th, ph)
        # every product and sum of a step rounds; the carried energy adds a step's change
        assert abs(float(e[j].item()) - ref) <= (j + 1) * (4 * nq + 128) * 2.0 ** -52 * float(np.abs(c).sum() + n)
    s.close(); ctx.close()
