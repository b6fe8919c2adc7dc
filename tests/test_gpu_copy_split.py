"""Copies into in-place stores whose buckets split, join or match the source's:
none, some and more hash bits than one work item counts, keys of one to four
words.  The copy holds the source's terms bit for bit, in source order inside
every bucket."""
import numpy as np
import pytest

from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms
from tests.test_gpu_inplace import INPLACE, _Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [30, 100, 150, 200])
@pytest.mark.parametrize("n,load,bits", [(1, 256, 0), (700, 16384, 0), (700, 16384, 6), (5000, 16384, 11), (5000, 256, 9),
                                         (5000, 64, 3), (20000, 128, 12)])
def test_copy_split(nq, n, load, bits):
    describe(nq, "store_copy", n=n, load_bucket_terms=load, bits=bits)
    x, z, c = random_terms(nq, n, n + nq)
    c[:: 7] = 0.25   # (keys tell the rows apart)
    n = len(c)
    ctx = iqcc.Context(0)
    per = 16
    with _Params(ctx, load_bucket_terms=load, inplace_bucket_terms=per):
        src = iqcc.Store(ctx, nq, 2 * n).load_numpy(x, z, c)
        dst = iqcc.Store(ctx, nq, max(per << bits, 3 * n) if bits else per, INPLACE) if bits or n <= per else None
        if dst is None:
            with _Params(ctx, inplace_bucket_terms=16384):
                dst = iqcc.Store(ctx, nq, 3 * n, INPLACE)
                iqcc.iqcc_store_copy(ctx.handle, src.handle, dst.handle)
        else:
            iqcc.iqcc_store_copy(ctx.handle, src.handle, dst.handle)
        got = dst.to_numpy()
        assert_same_terms(got, (x, z, c), f"copy {nq} {n} {load} {bits}")
        order = {k: i for i, k in enumerate(zip(*(map(tuple, a) for a in src.to_numpy()[:2])))}
        at = np.array([order[k] for k in zip(*(map(tuple, a) for a in got[:2]))])
        cap = max(per << bits, 3 * n) if bits else 16384
        buckets = 1 << max(0, round(np.log2(cap / per))) if bits else 1
        assert np.count_nonzero(np.diff(at) < 0) < max(buckets, 2)
        src.close(); dst.close()
    ctx.close()
