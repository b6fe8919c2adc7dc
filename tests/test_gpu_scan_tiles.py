"""Loads, copies and exports whose bucket counts take one tile of the offsets'
scan, several, and more than a workgroup adds up by itself."""
import numpy as np
import pytest

from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms
from tests.test_gpu_inplace import INPLACE, _Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [0, 9, 10, 11, 13, 20, 21])
@pytest.mark.parametrize("nq", [40, 100])
def test_scan_tiles(nq, bits):
    n = min(max((1 << bits) - 3, 5), 60_000)
    describe(nq, "scan tiles", bits=bits, n=n)
    x, z, c = random_terms(nq, n, n + nq + bits)
    n = len(c)
    ctx = iqcc.Context(0)
    with _Params(ctx, load_bucket_terms=1, inplace_bucket_terms=1):
        a = iqcc.Store(ctx, nq, 2 * n).load_numpy(x, z, c)
        assert_same_terms(a.to_numpy(), (x, z, c), "loaded")
        room = max(16 << bits, 2 * n)   # regions of at least 16 rows
        with _Params(ctx, inplace_bucket_terms=max(room >> bits, 1)):
            b = iqcc.Store(ctx, nq, room, INPLACE)
            iqcc.iqcc_store_copy(ctx.handle, a.handle, b.handle)
            assert_same_terms(b.to_numpy(), (x, z, c), "copied")
            b.load_numpy(x, z, c)
            assert_same_terms(b.to_numpy(), (x, z, c), "loaded in regions")
            assert b.count() == n
        a.close(); b.close()
    ctx.close()
