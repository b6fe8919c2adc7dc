"""Out-of-place steps with fewer bucket pairs than workgroups, as many, and on
both sides of the count up to which the rows are laid out in pair order; self
pairs (the identity); an output arena that is just too small."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms
from tests.test_gpu_inplace import _Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,n,load", [(20, 1, 256), (30, 900, 256), (30, 1030, 1), (30, 20_000, 1), (124, 20_000, 1),
                                       (30, 40_000, 1), (200, 700, 16)])
def test_dress_pairs(nq, n, load):
    ctx = iqcc.Context(0)
    x, z, c = random_terms(nq, n, nq + n)
    n = len(c)
    W = x.shape[1]
    with _Params(ctx, load_bucket_terms=load):
        a = iqcc.Store(ctx, nq, 2 * n).load_numpy(x, z, c)
    b = iqcc.Store(ctx, nq, 4 * n)
    for px, pz in (I.single_qubit_pauli(nq, "XZY"), (np.zeros(W, np.uint64), np.zeros(W, np.uint64))):
        describe(0, "dress pairs", nq=nq, n=n, load=load)
        iqcc.iqcc_dress(ctx.handle, a.handle, px, pz, 0.3, 1e-3, b.handle)
        ref = O.dress(nq, x, z, c, px, pz, 0.3, 1e-3)
        assert b.count() == len(ref[2])
        assert_same_terms(b.to_numpy(), ref, f"{nq} {n} {load}")
    a.close(); b.close(); ctx.close()


@pytest.mark.parametrize("load", [256, 1])
def test_dress_arena_too_small(load):
    ctx = iqcc.Context(0)
    x, z, c = random_terms(30, 30_000, 1)
    with _Params(ctx, load_bucket_terms=load):
        a = iqcc.Store(ctx, 30, 30_000).load_numpy(x, z, c)
    b, small, big = iqcc.Store(ctx, 30, 30_000), iqcc.Store(ctx, 30, 30_000), iqcc.Store(ctx, 30, 160_000)
    (px, pz), (qx, qz) = I.single_qubit_pauli(30, "XZY"), I.single_qubit_pauli(30, "IXY")
    iqcc.iqcc_dress(ctx.handle, a.handle, px, pz, 0.3, 1e-3, b.handle)   # 61,024 rows hold twice the input
    ref = O.dress(30, x, z, c, px, pz, 0.3, 1e-3)
    assert_same_terms(b.to_numpy(), ref, "fits")
    iqcc.iqcc_dress(ctx.handle, b.handle, qx, qz, 0.3, 1e-3, small.handle)   # not twice the grown sum
    with pytest.raises(iqcc.IqccError) as e:
        small.count()
    assert e.value.code == iqcc.IQCC_ERR_CAPACITY
    iqcc.iqcc_dress(ctx.handle, b.handle, qx, qz, 0.3, 1e-3, big.handle)   # the step's counters are clean again
    assert_same_terms(big.to_numpy(), O.dress(30, *ref, qx, qz, 0.3, 1e-3), "after an overflow")
    for st in (a, b, small, big):
        st.close()
    ctx.close()
