"""Calls of one thread and one context on different streams.

Steps that write different stores share nothing: a long step on one stream
with many short ones beside it, and a captured chain of steps replayed beside
eager ones, leave what the same calls leave one after another (the sums of a
step's workgroups lie in the memory of the store that it writes)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu

SHORT = 100      # short calls beside a long one


@pytest.fixture
def ctx():
    c = iqcc.Context(0)
    yield c
    c.close()


def long_step(ctx, src, p, dst, stream, **energy):
    """An out-of-place step with so small a stash that it takes milliseconds."""
    iqcc.iqcc_set_param(ctx.handle, "anti_cap", 16)
    iqcc.iqcc_dress(ctx.handle, src.handle, *p, 0.3, 0.0, dst.handle, stream=stream, **energy)
    iqcc.iqcc_set_param(ctx.handle, "anti_cap", 1024)


def test_short_steps_beside_a_long_one(ctx):
    nq = 40
    x, z, c = I.hamiltonian_dense(nq, 1)
    sx, sz, sc = random_terms(nq, 500, 1)
    p, q = I.single_qubit_pauli(nq, "XYZX"), I.single_qubit_pauli(nq, "ZXY")
    th, ph = I.qmf_angles(nq, np.random.default_rng(1))
    tht, pht = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    big = iqcc.Store(ctx, nq, 2 * len(c)).load_numpy(x, z, c)
    out = [iqcc.Store(ctx, nq, 2 * len(c)) for _ in range(2)]
    small = iqcc.Store(ctx, nq, 2 * len(sc)).load_numpy(sx, sz, sc)
    tail = [iqcc.Store(ctx, nq, 2 * len(sc)) for _ in range(SHORT)]
    rows = iqcc.iqcc_store_rows(small.handle)
    tapes = [torch.empty(rows, dtype=torch.int32, device="cuda") for _ in range(2)]
    home = iqcc.Store(ctx, nq, 8 * len(sc), iqcc.IQCC_STORE_INPLACE).load_numpy(sx, sz, sc)
    ref = O.dress(nq, x, z, c, *p, 0.3, 0.0)
    e_ref = O.qmf_energy(nq, *ref, th, ph)
    sref = O.dress(nq, sx, sz, sc, *q, 0.2, 0.0)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for it in range(3):
        describe(it, "short steps beside a long one", n=len(c), short=SHORT)
        e = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        long_step(ctx, big, p, out[0], a.cuda_stream)
        long_step(ctx, big, p, out[1], a.cuda_stream, theta=tht, phi=pht, energy=e[0])
        for k, t in enumerate(tail):
            if k % 3 == 0:
                iqcc.iqcc_dress(ctx.handle, small.handle, *q, 0.2, 0.0, t.handle, tht, pht, e[1], stream=b.cuda_stream)
            elif k % 3 == 1:
                iqcc.iqcc_dress(ctx.handle, small.handle, *q, 0.2, 0.0, t.handle, stream=b.cuda_stream)
            else:
                iqcc.iqcc_dress_taped(ctx.handle, small.handle, *q, 0.2, 0.0, t.handle, *tapes, stream=b.cuda_stream)
        iqcc.iqcc_dress_inplace(ctx.handle, home.handle, *q, 0.2 if it % 2 == 0 else -0.2, 0.0, stream=b.cuda_stream)
        torch.cuda.synchronize()
        for o in out:
            assert o.count() == len(ref[2])
            assert_same_terms(o.to_numpy(), ref)
        assert abs(e[0].item() - e_ref) <= 1e-10
        assert abs(e[1].item() - O.qmf_energy(nq, *sref, th, ph)) <= 1e-10
        for t in tail:
            assert t.count() == len(sref[2])
        assert_same_terms(tail[-1].to_numpy(), sref)
        assert home.count() == len(sref[2])
    for s in (big, small, home, *out, *tail):
        s.close()


def test_captured_chain_beside_eager_steps(ctx):
    """A chain of more steps than a context once had sets of words, captured and
    replayed several times beside eager steps on another stream."""
    nq = 24
    x, z, c = random_terms(nq, 4000, 2)
    p = I.single_qubit_pauli(nq, "XYZ")
    src = iqcc.Store(ctx, nq, 2 * len(c)).load_numpy(x, z, c)
    outs = [iqcc.Store(ctx, nq, 2 * len(c)) for _ in range(40)]
    others = [iqcc.Store(ctx, nq, 2 * len(c)) for _ in range(40)]
    ref = O.dress(nq, x, z, c, *p, 0.3, 1e-8)
    iqcc.iqcc_dress(ctx.handle, src.handle, *p, 0.3, 1e-8, others[0].handle)
    torch.cuda.synchronize()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(g, stream=s):
        for o in outs:
            iqcc.iqcc_dress(ctx.handle, src.handle, *p, 0.3, 1e-8, o.handle)
    b = torch.cuda.Stream()
    for it in range(4):
        describe(it, "captured chain beside eager steps", n=len(c))
        with torch.cuda.stream(s):
            g.replay()
        for o in others:
            iqcc.iqcc_dress(ctx.handle, src.handle, *p, 0.3, 1e-8, o.handle, stream=b.cuda_stream)
        torch.cuda.synchronize()
        for o in outs + others:
            assert o.count() == len(ref[2])
        assert_same_terms(outs[it].to_numpy(), ref)
        assert_same_terms(others[it].to_numpy(), ref)
    for o in (src, *outs, *others):
        o.close()
