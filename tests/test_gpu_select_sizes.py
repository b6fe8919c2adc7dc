"""Term limit at the edges of its passes: more terms equal in their first two
digits than one workgroup lists and just as many, ties among them, buckets
shorter and longer than a wavefront's slices, keys of one to four words.  The
kept set is compared with the oracle bit for bit."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_08883_amd import iqcc
from tests.gpu_util import assert_same_terms, describe
from tests.test_gpu_energy_sizes import random_terms

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = iqcc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("nq,n", [(30, 1), (30, 65), (30, 20000), (100, 8192), (100, 8193), (150, 20000), (200, 9001)])
@pytest.mark.parametrize("near", ["apart", "close", "close-ties"])
def test_term_limit_passes(ctx, nq, n, near):
    describe(nq, "truncate_top", n=n, near=near)
    rng = np.random.default_rng(n + nq)
    x, z, c = random_terms(nq, n, n + nq)
    n = len(c)
    if near != "apart":   # one value of the first two digits (22 bits), the others spread or equal
        low = rng.permutation(n) if near == "close" else rng.integers(0, max(n // 5, 1), n)
        c = 0.75 * (1.0 + low * 2.0 ** -45) * rng.choice([-1.0, 1.0], n)
    a = iqcc.Store(ctx, nq, n + 64).load_numpy(x, z, c)
    b = iqcc.Store(ctx, nq, n + 64)
    for keep in sorted({1, n // 2, max(n - 1, 1)}):
        iqcc.iqcc_truncate_top(ctx.handle, a.handle, keep, b.handle)
        assert b.count() == min(keep, n)
        assert_same_terms(b.to_numpy(), O.truncate_top(x, z, c, keep), f"{nq} {n} {near} {keep}")
    a.close(); b.close()
