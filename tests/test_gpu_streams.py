"""Calls of one thread and one context on different streams.

Steps that write different stores share nothing: a long step on one stream
with many short ones beside it, and a captured chain of steps replayed beside
eager ones, leave what the same calls leave one after another (the sums of a
step's workgroups lie in the memory of the store that it writes).  Sums over a
store that is only read give the same bits on many streams, captured and
replayed beside eager ones, and after all of these.  (Captured sums do not
overlap each other here: that they may not is documented.)"""
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


class Sums:
    """Every call that only reads stores, on a step of a small Hamiltonian."""

    def __init__(self, ctx, nq=40, n=3000):
        self.ctx = ctx
        x, z, c = random_terms(nq, n, nq + n)
        self.p = I.single_qubit_pauli(nq, "XYZ")
        self.th, self.ph = (torch.from_numpy(a).cuda() for a in I.qmf_angles(nq, np.random.default_rng(2)))
        self.h = iqcc.Store(ctx, nq, 2 * len(c)).load_numpy(x, z, c)
        self.out = iqcc.Store(ctx, nq, 2 * len(c))
        rows = iqcc.iqcc_store_rows(self.h.handle)
        self.tapes = [torch.empty(rows, dtype=torch.int32, device="cuda") for _ in range(2)]
        iqcc.iqcc_dress_taped(ctx.handle, self.h.handle, *self.p, 0.3, 0.0, self.out.handle, *self.tapes)
        self.lam = torch.linspace(-1, 1, iqcc.iqcc_store_rows(self.out.handle), dtype=torch.float64, device="cuda")
        self.oracle = O.qmf_energy(nq, x, z, c, self.th.cpu().numpy(), self.ph.cpu().numpy())
        torch.cuda.synchronize()

    def run(self, res, stream=None):
        """energy, allocation-free energy, energy of the anticommuting terms, dE/dtau and the
        cotangents of the step's input into res (a list of tensors)."""
        a = (self.ctx.handle, self.h.handle)
        iqcc.iqcc_qmf_energy(*a, self.th, self.ph, res[0], stream=stream)
        iqcc.iqcc_qmf_energy_noalloc(*a, self.th, self.ph, res[1], stream=stream)
        iqcc.iqcc_qmf_energy_anti(*a, *self.p, self.th, self.ph, res[2], stream=stream)
        iqcc.iqcc_dress_backward(*a, *self.p, 0.3, *self.tapes, self.lam, res[4], res[3], stream=stream)

    def buffers(self):
        d = dict(dtype=torch.float64, device="cuda")
        return [torch.full((), 7.0, **d) for _ in range(4)] + [torch.full((iqcc.iqcc_store_rows(self.h.handle),), 7.0, **d)]

    def close(self):
        self.h.close()
        self.out.close()


def same_bits(a, b):
    return all(torch.equal(u, v) for u, v in zip(a, b))


def test_sums_on_many_streams(ctx):
    """More streams than have sums of their own, each a few calls ahead of the
    others; streams beyond those one after another (see the header)."""
    t = Sums(ctx)
    ref = t.buffers()
    t.run(ref)
    torch.cuda.synchronize()
    assert abs(ref[0].item() - t.oracle) <= 1e-10 and ref[0].item() == ref[1].item()
    streams = [torch.cuda.Stream() for _ in range(20)]
    handles = {s.cuda_stream for s in streams}
    describe(0, "sums on many streams", n=t.h.count(), streams=len(handles))
    for it in range(3):
        got = {s: [t.buffers() for _ in range(12)] for s in streams}
        torch.cuda.synchronize()
        for k in range(12):
            for s in streams[:12]:
                a = (ctx.handle, t.h.handle)
                r = got[s][k]
                iqcc.iqcc_qmf_energy(*a, t.th, t.ph, r[0], stream=s.cuda_stream)
                iqcc.iqcc_qmf_energy_anti(*a, *t.p, t.th, t.ph, r[2], stream=s.cuda_stream)
                iqcc.iqcc_dress_backward(*a, *t.p, 0.3, *t.tapes, t.lam, r[4], r[3], stream=s.cuda_stream)
        torch.cuda.synchronize()
        for s in streams[:12]:
            for r in got[s]:
                assert same_bits(r[:1] + r[2:], ref[:1] + ref[2:])
        for s in streams[12:]:
            t.run(got[s][0], s.cuda_stream)
            torch.cuda.synchronize()
            assert same_bits(got[s][0], ref)
    t.close()


def test_captured_sums(ctx):
    t = Sums(ctx)
    ref, cap, eager = t.buffers(), t.buffers(), t.buffers()
    t.run(ref)
    t.run(cap)
    torch.cuda.synchronize()
    g, s, b = torch.cuda.CUDAGraph(), torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.graph(g, stream=s):
        t.run(cap)
    for it in range(6):
        describe(it, "captured sums")
        for r in cap + eager:
            r.fill_(7.0)
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            g.replay()
        for _ in range(40):
            a = (ctx.handle, t.h.handle)
            iqcc.iqcc_qmf_energy(*a, t.th, t.ph, eager[0], stream=b.cuda_stream)
            iqcc.iqcc_qmf_energy_anti(*a, *t.p, t.th, t.ph, eager[2], stream=b.cuda_stream)
            iqcc.iqcc_dress_backward(*a, *t.p, 0.3, *t.tapes, t.lam, eager[4], eager[3], stream=b.cuda_stream)
        torch.cuda.synchronize()
        iqcc.iqcc_qmf_energy_noalloc(ctx.handle, t.h.handle, t.th, t.ph, eager[1])
        torch.cuda.synchronize()
        assert same_bits(cap, ref)
        assert same_bits(eager, ref)
    t.close()
