"""Loading a store over the forms of its three passes: buckets counted in LDS or
in global counters, one or several wavefronts per bucket, remainders, one
bucket, buckets of one term -- the same rows for any input order, the same
terms, ascending keys within a bucket."""
import numpy as np
import pytest

from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,n,bucket,flags", [
    (30, 0, 256, 0), (30, 1, 256, 0), (40, 257, 256, 0), (64, 5000, 256, 0), (64, 5000, 1, 0), (70, 9000, 16384, 0),
    (124, 70_000, 64, 0), (124, 70_000, 65, 0), (150, 3000, 3, 0), (200, 1000, 500, 0),
    (40, 6000, 256, iqcc.IQCC_STORE_INPLACE), (124, 300, 256, iqcc.IQCC_STORE_INPLACE)])
def test_load_sizes(nq, n, bucket, flags):
    ctx = iqcc.Context(0)
    iqcc.iqcc_set_param(ctx.handle, "load_bucket_terms", bucket)
    x, z, c = random_terms(nq, n, nq + n + bucket)
    n = len(c)
    rng = np.random.default_rng(1)
    got = []
    for order in (np.arange(n), rng.permutation(n)):
        describe(0, "load sizes", nq=nq, n=n, bucket=bucket, flags=flags)
        s = iqcc.Store(ctx, nq, max(16 * n, 64), flags).load_numpy(x[order], z[order], c[order])
        got.append(s.to_numpy())
        s.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    assert_same_terms(got[0], (x, z, c))
    if bucket == 16384 and n:       # one bucket: the whole store in ascending key order
        gx, gz, _ = got[0]
        keys = [tuple(r) for r in np.concatenate([gx[:, ::-1], gz[:, ::-1]], 1).tolist()]
        assert keys == sorted(keys)
    ctx.close()
