"""In-place steps (Eq. 5) over the item sizes of the step: one pair per item
where there are fewer pairs than waves, several where buckets are many and
small, one bucket, an entangler whose hash bits vanish (self pairs, here the
identity), and one workgroup's worth of counters read back after every step."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,n,max_terms", [(20, 1, 16), (24, 300, 4000), (30, 3000, 300_000), (70, 5000, 2_000_000),
                                            (124, 20_000, 6_000_000), (150, 700, 40_000), (200, 900, 200_000)])
def test_inplace_items(nq, n, max_terms):
    ctx = iqcc.Context(0)
    x, z, c = random_terms(nq, n, 7 * nq + n)
    rng = np.random.default_rng(nq)
    th, ph = I.qmf_angles(nq, rng)
    tht, pht = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    s = iqcc.Store(ctx, nq, max_terms, iqcc.IQCC_STORE_INPLACE).load_numpy(x, z, c)
    e = torch.zeros(4, dtype=torch.float64, device="cuda")
    W = x.shape[1]
    ents = [I.single_qubit_pauli(nq, "XYZ"), (np.zeros(W, np.uint64), np.zeros(W, np.uint64)),
            I.single_qubit_pauli(nq, "IZXXY"), I.single_qubit_pauli(nq, "XYZ")]
    for j, (px, pz) in enumerate(ents):
        describe(j, "inplace items", nq=nq, n=n, max_terms=max_terms)
        iqcc.iqcc_dress_inplace(ctx.handle, s.handle, px, pz, 0.2 + 0.1 * j, 1e-3, tht, pht,
                                e[j - 1:j] if j else None, e[j:j + 1])
        raw = len(O.dress_raw(nq, x, z, c, px, pz, 0.2 + 0.1 * j)[2]) - len(c)
        before = {(a.tobytes(), b.tobytes()) for a, b in zip(x, z)}
        x, z, c = O.dress(nq, x, z, c, px, pz, 0.2 + 0.1 * j, 1e-3)
        new = sum((a.tobytes(), b.tobytes()) not in before for a, b in zip(x, z))
        assert_same_terms(s.to_numpy(), (x, z, c), f"step {j}")
        assert s.count() == len(c)
        assert iqcc.iqcc_store_stats(ctx.handle, s.handle) == (raw, new)
        ref = O.qmf_energy(nq, x, z, c, th, ph)
        assert abs(float(e[j].item()) - ref) <= (j + 1) * (4 * nq + 128) * 2.0 ** -52 * float(np.abs(c).sum() + 1)
    s.close(); ctx.close()
