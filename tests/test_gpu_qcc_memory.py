"""Working memory of flip sets and of an iteration: given back after a large
Hamiltonian, in whatever order small and large ones come, and the same results."""
import numpy as np
import pytest
import torch

from oracle import qcc as Q
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


def test_work_memory_is_given_back():
    ctx = iqcc.Context(0)
    nq, n = 40, 40_000_000      # 2^27 table entries: more than 1 GiB
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randint(0, 1 << 12, (1, n), dtype=torch.int64, device="cuda", generator=g)
    z = torch.arange(n, device="cuda").reshape(1, n).contiguous()
    big = iqcc.Store(ctx, nq, n)
    iqcc.iqcc_store_load(ctx.handle, big.handle, x, z, torch.ones(n, dtype=torch.float64, device="cuda"))
    sx, sz, sc = random_terms(12, 300, 5)
    small = iqcc.Store(ctx, 12, 4096).load_numpy(sx, sz, sc)
    ref = Q.flip_sets(sx, 12)
    want = len([v for v in torch.unique(x).tolist() if v])
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for it in range(3):
        describe(it, "flip sets of a large and a small Hamiltonian", n=n)
        assert len(iqcc.iqcc_flip_sets(ctx.handle, big.handle, 12)) == want
        assert free - torch.cuda.mem_get_info()[0] <= 64 << 20
        assert np.array_equal(iqcc.iqcc_flip_sets(ctx.handle, small.handle, 12), ref)
    big.close(); small.close(); ctx.close()


def test_iterations_of_growing_size():
    """One context, blocks that grow between calls: as on a fresh context."""
    ctx = iqcc.Context(0)
    for nq, n in ((10, 20), (30, 3000), (12, 5), (40, 20_000), (70, 500)):
        x, z, c = random_terms(nq, n, nq)
        th, ph = (torch.from_numpy(a).cuda() for a in I.qmf_angles(nq, np.random.default_rng(nq)))
        got = []
        for c_ in (ctx, iqcc.Context(0)):
            h = iqcc.Store(c_, nq, 4 * len(c) + 64).load_numpy(x, z, c)
            spare = iqcc.Store(c_, nq, 4 * len(c) + 64)
            describe(nq, "iterations of growing size", n=len(c))
            r = iqcc.iqcc_qcc_iteration(c_.handle, h, spare, th, ph, 6, 2, 1e-9)
            got.append((r["n_candidates"], r["sel_x"].tolist(), r["sel_z"].tolist(), r["energy"].tolist()))
            h.close(); spare.close()
            if c_ is not ctx:
                c_.close()
        assert got[0][:3] == got[1][:3] and np.allclose(got[0][3], got[1][3], rtol=1e-13, atol=1e-13)
    ctx.close()
