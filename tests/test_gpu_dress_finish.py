"""The finish of an out-of-place step (Eq. 5): counters, error flags and the
energy are written by the workgroup that arrives last, from words that are
reset for the next step.  A step that runs out of rows reports it, its output
is refused by the next step, and a step after them is right; the energy table's
build fits the smallest stash; grids of one and of many workgroups per CU; the
energy summed apart."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


def test_overflow_then_valid_step():
    ctx = iqcc.Context(0)
    nq = 40
    x, z, c = random_terms(nq, 1000, 3)
    th, ph = (torch.from_numpy(a).cuda() for a in I.qmf_angles(nq, np.random.default_rng(1)))
    px, pz = I.single_qubit_pauli(nq, "XYZ")
    small = iqcc.Store(ctx, nq, 100).load_numpy(x, z, c)      # 1224 rows: a step of 1000 terms reserves 2000
    a, b = iqcc.Store(ctx, nq, 100), iqcc.Store(ctx, nq, 100)
    e = torch.zeros(1, dtype=torch.float64, device="cuda")
    describe(0, "dress into a full arena", n=len(c))
    iqcc.iqcc_dress(ctx.handle, small.handle, px, pz, 0.3, 0.0, a.handle, th, ph, e)
    with pytest.raises(iqcc.IqccError) as err:
        a.count()
    assert err.value.code == iqcc.IQCC_ERR_CAPACITY
    iqcc.iqcc_dress(ctx.handle, a.handle, px, pz, 0.3, 0.0, b.handle, th, ph, e)
    with pytest.raises(iqcc.IqccError) as err:
        b.count()
    assert err.value.code == iqcc.IQCC_ERR_CAPACITY
    h, out = iqcc.Store(ctx, nq, 1000).load_numpy(x, z, c), iqcc.Store(ctx, nq, 1000)
    ref = O.dress(nq, x, z, c, px, pz, 0.3, 0.0)
    for _ in range(40):      # more steps than there are sets of words
        iqcc.iqcc_dress(ctx.handle, h.handle, px, pz, 0.3, 0.0, out.handle, th, ph, e)
    assert_same_terms(out.to_numpy(), ref)
    assert abs(float(e.item()) - O.qmf_energy(nq, *ref, th.cpu().numpy(), ph.cpu().numpy())) <= 1e-10
    for s in (small, a, b, h, out):
        s.close()
    ctx.close()


@pytest.mark.parametrize("nq,n,knobs", [(9, 1, {}), (40, 3000, {"anti_cap": 16}), (40, 3000, {"grid_per_cu": 16, "anti_cap": 64}),
                                        (100, 3000, {"grid_per_cu": 1}), (124, 2000, {"fuse_energy": 0}),
                                        (200, 900, {"anti_cap": 16}), (256, 900, {})])
def test_dress_finish(nq, n, knobs):
    ctx = iqcc.Context(0)
    for k, v in knobs.items():
        iqcc.iqcc_set_param(ctx.handle, k, v)
    x, z, c = random_terms(nq, n, 11 * nq + n)
    th, ph = I.qmf_angles(nq, np.random.default_rng(nq))
    tht, pht = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    a, b = iqcc.Store(ctx, nq, 8 * n).load_numpy(x, z, c), iqcc.Store(ctx, nq, 8 * n)
    e = torch.zeros(1, dtype=torch.float64, device="cuda")
    for j, word in enumerate(("XYZ", "IZXXY")):
        px, pz = I.single_qubit_pauli(nq, word)
        describe(j, "dress finish", nq=nq, n=n, knobs=knobs)
        if j == 0:
            iqcc.iqcc_dress(ctx.handle, a.handle, px, pz, 0.4, 1e-3, b.handle, tht, pht, e)
        else:
            iqcc.iqcc_dress_energy_update(ctx.handle, a.handle, px, pz, 0.4, 1e-3, b.handle, tht, pht, e, e)
        raw = len(O.dress_raw(nq, x, z, c, px, pz, 0.4)[2]) - len(c)
        before = {(p.tobytes(), q.tobytes()) for p, q in zip(x, z)}
        x, z, c = O.dress(nq, x, z, c, px, pz, 0.4, 1e-3)
        new = sum((p.tobytes(), q.tobytes()) not in before for p, q in zip(x, z))
        assert_same_terms(b.to_numpy(), (x, z, c), f"step {j}")
        assert iqcc.iqcc_store_stats(ctx.handle, b.handle) == (raw, new)
        ref = O.qmf_energy(nq, x, z, c, th, ph)
        assert abs(float(e.item()) - ref) <= (j + 1) * (4 * nq + 128) * 2.0 ** -52 * float(np.abs(c).sum() + 1)
        a, b = b, a
    a.close(); b.close(); ctx.close()
