"""The allocation-free energy over all values of the knob of its grid: none is
refused, and each gives the energy of the allocating call bit for bit."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import describe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [8, 40])
def test_noalloc_grids(nq):
    ctx = iqcc.Context(0)
    x, z, c = I.hamiltonian_dense(nq, 0)
    th, ph = I.qmf_angles(nq, np.random.default_rng(nq))
    tht, pht = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    s = iqcc.Store(ctx, nq, 2 * len(c)).load_numpy(x, z, c)
    ref = O.qmf_energy(nq, x, z, c, th, ph)
    for g in (1, 2, 16, 32):
        describe(g, "noalloc grid", nq=nq, n=len(c))
        iqcc.iqcc_set_param(ctx.handle, "energy_grid_per_cu", g)
        a = iqcc.iqcc_qmf_energy_noalloc(ctx.handle, s.handle, tht, pht).item()
        assert a == iqcc.iqcc_qmf_energy(ctx.handle, s.handle, tht, pht).item()
        assert abs(a - ref) <= 1e-10
    s.close()
    ctx.close()
