"""In-place stores with far more buckets than terms: most of a workgroup's
buckets, of its groups and of a term range are empty.  Energy, angle gradient
and screening against the oracle, and in-place steps whose items are many empty
pairs, or as many as there are waves."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import describe
from tests.test_gpu_dis_sizes import candidates
from tests.test_gpu_energy_sizes import random_terms
from tests.test_gpu_inplace_items import test_inplace_items as inplace_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,n,max_terms,n_cand", [
    (40, 0, 1 << 22, 3), (40, 1, 1 << 20, 1), (40, 700, 1 << 24, 300), (40, 20_000, 1 << 25, 7),
    (100, 700, 1 << 24, 40), (150, 300, 1 << 22, 33), (250, 300, 1 << 22, 2)])
def test_sparse_store(nq, n, max_terms, n_cand):
    ctx = iqcc.Context(0)
    x, z, c = random_terms(nq, n, nq + n)
    th, ph = I.qmf_angles(nq, np.random.default_rng(nq))
    tht, pht = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    cx, cz = candidates(nq, n_cand, nq + n_cand)
    s = iqcc.Store(ctx, nq, max_terms, iqcc.IQCC_STORE_INPLACE).load_numpy(x, z, c)
    describe(0, "sparse store", nq=nq, n=n, max_terms=max_terms, n_cand=n_cand)
    e = iqcc.iqcc_qmf_energy(ctx.handle, s.handle, tht, pht).item()
    dt, dp = iqcc.iqcc_qmf_energy_backward(ctx.handle, s.handle, tht, pht)
    g = iqcc.iqcc_dis_gradients(ctx.handle, s.handle, tht, pht, iqcc.to_device_words(cx), iqcc.to_device_words(cz))
    # rounding: nq factors, twelve ratios or a division a term, sums of depth below 256
    tol = 3 * (4 * nq + 256) * 2.0 ** -53 * float(np.abs(c).sum())
    if n == 0:
        assert e == 0.0 and not dt.any() and not dp.any() and not g.any()
    else:
        assert abs(e - O.qmf_energy(nq, x, z, c, th, ph)) <= tol
        rt, rp = O.qmf_grad_angles(nq, x, z, c, th, ph)
        assert np.abs(dt.cpu().numpy() - rt).max() <= tol and np.abs(dp.cpu().numpy() - rp).max() <= tol
        assert np.abs(g.cpu().numpy() - O.dis_gradients(nq, x, z, c, th, ph, cx, cz)).max() <= tol
    s.close()
    ctx.close()


@pytest.mark.parametrize("nq,n,max_terms", [(40, 2000, 1 << 24), (40, 1, 1 << 20), (100, 60_000, 1 << 24),
                                            (150, 900, 1 << 22), (250, 3000, 1 << 21)])
def test_sparse_inplace_steps(nq, n, max_terms):
    inplace_steps(nq, n, max_terms)


@pytest.mark.parametrize("nq,n,max_terms", [(40, 60_000, 1 << 22), (100, 300_000, 1 << 22), (170, 300_000, 9_000_000),
                                            (250, 300_000, 9_000_000), (250, 30_000, 1 << 22)])
@pytest.mark.parametrize("energy", [False, True])
def test_items_fit_the_stash(nq, n, max_terms, energy):
    """Wide keys leave little stash: items are not made so large, to be few, that
    their anticommuting terms have to go to the store's pool."""
    ctx = iqcc.Context(0)
    g = torch.Generator(device="cuda").manual_seed(nq)
    W = (nq + 63) // 64
    x, z = (torch.randint(0, 1 << (nq % 64 or 62), (W, n), dtype=torch.int64, device="cuda", generator=g) for _ in range(2))
    c = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    th, ph = (torch.from_numpy(a).cuda() for a in I.qmf_angles(nq, np.random.default_rng(nq)))
    s = iqcc.Store(ctx, nq, max_terms, iqcc.IQCC_STORE_INPLACE)
    iqcc.iqcc_store_load(ctx.handle, s.handle, x, z, c)
    assert len(torch.unique(x[0])) == n      # distinct keys
    p = I.single_qubit_pauli(nq, "XYZ")
    e = torch.zeros(1, dtype=torch.float64, device="cuda")
    for step in range(4):                    # the second step finds every image: two thirds anticommute
        describe(step, "items fit the stash", nq=nq, n=n, max_terms=max_terms, energy=energy)
        iqcc.iqcc_dress_inplace(ctx.handle, s.handle, *p, 0.1, 0.0, *((th, ph, None, e) if energy else ()))
        assert iqcc.iqcc_store_inplace_stats(ctx.handle, s.handle)["relocated"] == 0
    s.count()
    s.close()
    ctx.close()
