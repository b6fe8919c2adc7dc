"""The output store of a term limit: its rows are the selection's scratch (the
keys of equal terms too, so the call allocates nothing), its bucket regions are
gone afterwards, and a call that is refused leaves it as it was."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu
IP = iqcc.IQCC_STORE_INPLACE


@pytest.fixture
def ctx():
    c = iqcc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("nq,n,keep", [(30, 1000, 1), (40, 70_000, 34_567), (100, 70_000, 69_999), (150, 9000, 4000),
                                       (200, 9000, 8200)])
def test_equal_terms_into_an_inplace_store(ctx, nq, n, keep):
    x, z, c = random_terms(nq, n, nq + n)
    c = np.sign(c) * 0.25
    a = iqcc.Store(ctx, nq, 2 * n, IP).load_numpy(x, z, c)
    out = iqcc.Store(ctx, nq, 2 * n, IP).load_numpy(x[:10], z[:10], c[:10])
    describe(nq, "term limit of equal terms", n=n, keep=keep)
    ref = O.truncate_top(x, z, c, keep)
    for _ in range(2):
        iqcc.iqcc_truncate_top(ctx.handle, a.handle, keep, out.handle)
        assert out.count() == keep
        assert_same_terms(out.to_numpy(), ref)
    p = I.single_qubit_pauli(nq, "XYZ")
    with pytest.raises(iqcc.IqccError) as e:     # no bucket regions any more
        iqcc.iqcc_dress_inplace(ctx.handle, out.handle, *p, 0.3, 0.0)
    assert e.value.code == iqcc.IQCC_ERR_INVALID_ARG
    home = iqcc.Store(ctx, nq, 2 * n, IP)        # as many buckets as `out` had regions
    iqcc.iqcc_store_copy(ctx.handle, out.handle, home.handle)
    iqcc.iqcc_dress_inplace(ctx.handle, home.handle, *p, 0.3, 0.0)
    assert_same_terms(home.to_numpy(), O.dress(nq, *ref, *p, 0.3, 0.0))
    for s in (a, out, home):
        s.close()


def test_invalid_input_leaves_the_output(ctx):
    nq = 40
    x, z, c = random_terms(nq, 1000, 3)
    p = I.single_qubit_pauli(nq, "XYZ")
    small = iqcc.Store(ctx, nq, 100).load_numpy(x, z, c)      # 1224 rows: a step of 1000 terms reserves 2000
    bad = iqcc.Store(ctx, nq, 100)
    iqcc.iqcc_dress(ctx.handle, small.handle, *p, 0.3, 0.0, bad.handle)
    out = iqcc.Store(ctx, nq, 4000, IP).load_numpy(x, z, c)
    for keep in (0, 10, 5000):
        describe(keep, "term limit of an invalid store")
        with pytest.raises(iqcc.IqccError) as e:
            iqcc.iqcc_truncate_top(ctx.handle, bad.handle, keep, out.handle)
        assert e.value.code == iqcc.IQCC_ERR_CAPACITY
        assert_same_terms(out.to_numpy(), (x, z, c))
    iqcc.iqcc_dress_inplace(ctx.handle, out.handle, *p, 0.3, 0.0)   # its regions are still there
    assert_same_terms(out.to_numpy(), O.dress(nq, x, z, c, *p, 0.3, 0.0))
    for s in (small, bad, out):
        s.close()

