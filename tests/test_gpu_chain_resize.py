"""A differentiable chain run again with amplitudes under which its stores, sized
by the first run, are too small: the run notices and sizes them anew, and energy
and gradients equal those of a fresh chain and of the oracle; a run that fits
again takes them as they are."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from paper_2603_08883_amd.autograd import DressingChain, qmf_chain_energy
from tests.gpu_util import describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


def test_chain_outgrows_its_stores():
    ctx = iqcc.Context(0)
    nq, eps = 40, 1e-3
    x, z, c = random_terms(nq, 4000, 17)
    ents = [I.single_qubit_pauli(nq, w) for w in ("XYZ", "IIXYZ", "IZXIXY", "YXXXI", "IIIIZZXY")]
    th, ph = I.qmf_angles(nq, np.random.default_rng(5))
    chain = DressingChain(ctx, nq, x, z, c, ents, eps)

    def step(ch, taus):
        t = [torch.from_numpy(a.copy()).cuda().requires_grad_(True) for a in (th, ph, taus)]
        e = qmf_chain_energy(*t, ch)
        e.backward()
        return [e.detach().cpu().numpy()] + [a.grad.cpu().numpy() for a in t]

    small, big = np.full(5, 1e-6), np.array([0.4, -0.7, 0.9, 0.3, -0.5])
    for k, taus in enumerate((small, big, small, big)):
        describe(k, "chain resize", taus=taus.tolist())
        got = step(chain, taus)
        fresh = DressingChain(ctx, nq, x, z, c, ents, eps)
        ref = step(fresh, taus)
        caps = list(chain.caps)
        for a, b in zip(got, ref):
            assert np.abs(a - b).max() <= 1e-11 * (1 + np.abs(b).max())
        fx, fz, fc = O.chain(nq, x, z, c, ents, taus, eps)
        assert chain.stores[-1].count() == len(fc)
        assert abs(float(got[0]) - O.qmf_energy(nq, fx, fz, fc, th, ph)) <= 1e-10
        fresh.close()
        if k == 0:
            first = caps
    assert caps[-1] > first[-1], "the second run did not outgrow the first one's stores"
    chain.close(); ctx.close()
