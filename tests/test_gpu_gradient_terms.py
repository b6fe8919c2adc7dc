"""Angle gradients (derivative of Eq. 3) of more than 2^24 terms in one
workgroup: the digit sums pass their carries on before they leave 32 bits.

No call makes so large a bucket (a load ranks each bucket's terms), so the test
takes a loaded store, whose rows lie one after another, and writes "one bucket
of all rows" into the bucket table in its memory."""
import numpy as np
import pytest
import torch

from paper_2603_08883_amd import inputs as I
from paper_2603_08883_amd import iqcc
from tests.gpu_util import describe

pytestmark = pytest.mark.gpu

N = (1 << 24) + (1 << 20) + 77


def one_bucket(s, n, max_terms):
    mcap = int(np.ceil(np.log2(max_terms // 16 + 1))) + 1
    words = s.mem.view(torch.int64)
    cnt = (256 + 8 * (1 << mcap)) // 8           # header, off
    m = int(s.mem.view(torch.int32)[4].item())   # bucket bits
    assert 0 <= m <= mcap
    total = int(words[cnt:cnt + (1 << m)].sum().item())
    assert int(words[0].item()) == n and total == n and int(words[256 // 8].item()) == 0
    words[cnt] = n
    s.mem.view(torch.int32)[4] = 0


@pytest.mark.parametrize("nq", [40, 100, 170, 250])
def test_equal_terms_of_one_workgroup(nq):
    """Z strings near a pole: every product is exactly 1, every digit of c is 127."""
    ctx = iqcc.Context(0)
    W = (nq + 63) // 64
    z = torch.zeros((W, N), dtype=torch.int64, device="cuda")
    z[0] = torch.arange(1, N + 1, device="cuda")
    c = torch.full((N,), 2.0 - 2.0 ** -52, dtype=torch.float64, device="cuda")
    th = torch.full((nq,), 1e-9, dtype=torch.float64, device="cuda")
    ph = torch.full((nq,), 0.3, dtype=torch.float64, device="cuda")
    s = iqcc.Store(ctx, nq, N)
    iqcc.iqcc_store_load(ctx.handle, s.handle, torch.zeros_like(z), z, c)
    one_bucket(s, N, N)
    describe(0, "equal terms of one workgroup", nq=nq, n=N)
    dt, dp = iqcc.iqcc_qmf_energy_backward(ctx.handle, s.handle, th, ph)
    count = np.array([int(((z[0] >> q) & 1).sum().item()) if q < 63 else 0 for q in range(nq)], dtype=np.float64)
    ref = -np.sin(1e-9) * count * (2.0 - 2.0 ** -52)
    # the sum's value is rounded while its digits are joined, then three products
    assert np.abs(dt.cpu().numpy() - ref).max() <= 8 * 2.0 ** -53 * np.abs(ref).max()
    assert not dp.any()
    s.close()
    ctx.close()


@pytest.mark.parametrize("nq", [40, 100])
def test_mixed_terms_of_one_workgroup(nq):
    """The same rows in one bucket and in many: the same exact sums, rounded once
    per workgroup."""
    ctx = iqcc.Context(0)
    W = (nq + 63) // 64
    g = torch.Generator(device="cuda").manual_seed(nq)
    x, z = (torch.randint(0, 1 << 36, (W, N), dtype=torch.int64, device="cuda", generator=g) for _ in range(2))
    x[0] = torch.arange(N, device="cuda") ^ (x[0] & ~((1 << 25) - 1))       # distinct in the low bits
    c = torch.randn(N, dtype=torch.float64, device="cuda", generator=g)
    th, ph = (torch.from_numpy(a).cuda() for a in I.qmf_angles(nq, np.random.default_rng(nq)))
    s = iqcc.Store(ctx, nq, N)
    iqcc.iqcc_store_load(ctx.handle, s.handle, x, z, c)
    many = iqcc.iqcc_qmf_energy_backward(ctx.handle, s.handle, th, ph)
    one_bucket(s, N, N)
    describe(0, "mixed terms of one workgroup", nq=nq, n=N)
    one = iqcc.iqcc_qmf_energy_backward(ctx.handle, s.handle, th, ph)
    scale = (c * 1.0).abs().sum().item()
    for a, b in zip(one, many):
        assert torch.isfinite(a).all()
        # one rounding per workgroup and sum of 256, divisions, three products:
        # each within an ulp of at most the sum of |c|
        assert (a - b).abs().max().item() <= 3 * 300 * 2.0 ** -53 * scale
    s.close()
    ctx.close()
