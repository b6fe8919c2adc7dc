"""The device side of an iteration (flip sets, candidates, selection, the two
anticommuting sums) at its edges: one term, one candidate, fewer candidates
than asked for, none asked for, several words, gradients that are exactly zero
(never taken) and equal ones (canonical key order), and the single-generator
sums against the oracle's."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from oracle import qcc as Q
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,n,w_max,n_select,angles", [
    (6, 1, 6, 3, "random"), (10, 40, 4, 0, "random"), (12, 300, 3, 5, "random"), (8, 200, 8, 40, "equal"),
    (20, 1500, 5, 4, "poles"), (70, 400, 30, 3, "random"), (130, 200, 60, 2, "random"), (10, 3, 1, 100, "random")])
def test_iteration_edges(nq, n, w_max, n_select, angles):
    ctx = iqcc.Context(0)
    x, z, c = random_terms(nq, n, 13 * nq + n)
    th, ph = I.qmf_angles(nq, np.random.default_rng(nq))
    if angles == "equal":       # qubits alike: many gradients of equal size
        th[:], ph[:] = 0.7, 0.4
        c = np.sign(c)
    if angles == "poles":
        th = np.where(np.arange(nq) % 2 == 0, 0.0, th)
    tht, pht = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    describe(0, "iteration edges", nq=nq, n=len(c), w_max=w_max, n_select=n_select, angles=angles)
    room = min(4 ** nq, max(len(c), 16) << n_select)      # a step at most doubles the terms
    h = iqcc.Store(ctx, nq, room).load_numpy(x, z, c)
    spare = iqcc.Store(ctx, nq, room)
    F = Q.flip_sets(x, w_max)
    assert np.array_equal(iqcc.iqcc_flip_sets(ctx.handle, h.handle, w_max), F)
    gx, gz = Q.dis_generators(F)
    s = float(np.abs(c).sum())
    tol = (8 * nq + 256) * 2.0 ** -53 * s
    if len(gx):
        g = O.dis_gradients(nq, x, z, c, th, ph, gx, gz)
        for k in {0, len(gx) // 2, len(gx) - 1}:
            b = iqcc.iqcc_qmf_energy_anti(ctx.handle, h.handle, gx[k], gz[k], tht, pht).item()
            assert abs(b - Q.energy_anti(nq, x, z, c, gx[k], gz[k], th, ph)) <= tol
    got = iqcc.iqcc_qcc_iteration(ctx.handle, h, spare, tht, pht, w_max, n_select, 1e-9)
    assert got["n_candidates"] == len(gx)
    assert abs(got["energy"][0] - O.qmf_energy(nq, x, z, c, th, ph)) <= tol
    taken = len(got["sel_g"])
    if n_select and len(gx):
        # in rank order with the gradients of these very candidates; where two
        # are equal within rounding either may come first, but never a smaller
        # one, and exact zeros are not taken
        order = np.sort(np.abs(g))[::-1]
        assert taken <= min(n_select, len(gx))
        assert np.abs(np.abs(got["sel_g"]) - order[:taken]).max(initial=0.0) <= tol
        if taken < min(n_select, len(gx)):
            assert order[taken] <= tol
        seen = {tuple(a) + tuple(b): v for a, b, v in zip(gx.tolist(), gz.tolist(), g)}
        keys = [tuple(a) + tuple(b) for a, b in zip(got["sel_x"].tolist(), got["sel_z"].tolist())]
        assert len(set(keys)) == taken
        for k, v in zip(keys, got["sel_g"]):
            assert abs(seen[k] - v) <= tol
        for i in range(1, taken):
            a, b = got["sel_g"][i - 1], got["sel_g"][i]
            assert abs(a) >= abs(b)
            if abs(a) == abs(b):
                assert O.canonical(*(np.array([u, v], np.uint64) for u, v in (
                    (got["sel_x"][i - 1], got["sel_x"][i]), (got["sel_z"][i - 1], got["sel_z"][i]))),
                    np.array([0.0, 1.0]))[2].tolist() == [0.0, 1.0]
        # the closed-form steps of those generators
        for k in range(taken):
            px, pz = got["sel_x"][k], got["sel_z"][k]
            b = Q.energy_anti(nq, x, z, c, px, pz, th, ph)
            cc = O.dis_gradients(nq, x, z, c, th, ph, px[None], pz[None])[0]
            if np.hypot(b, cc) > 1e-6 * s:
                assert abs(got["sel_tau"][k] - np.arctan2(-cc, -b)) <= 1e-8
            x, z, c = O.dress(nq, x, z, c, px, pz, float(got["sel_tau"][k]), 1e-9)
            assert abs(got["energy"][k + 1] - O.qmf_energy(nq, x, z, c, th, ph)) <= 1e-9 * (1 + s)
        assert h.count() == len(c)
    else:
        assert taken == 0
    h.close(); spare.close(); ctx.close()
