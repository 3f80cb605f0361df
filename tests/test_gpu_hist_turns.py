"""The histograms whose lanes start with different subspaces, and the rule that sends large updates to the indices sorted by
cluster: against the oracle, for word counts that the turns do not divide and clusters whose codes are all alike."""
from __future__ import annotations

import numpy as np
import pytest

from _util import u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", [0, 2, 3])
@pytest.mark.parametrize("N,M,K", [(1, 4, 1), (63, 12, 3), (1025, 20, 7), (5000, 16, 300), (4097, 32, 65), (3000, 64, 5),
                                   (2049, 28, 129), (70_001, 8, 700), (40_003, 24, 50), (9001, 40, 33), (5003, 48, 90), (30_001, 6, 40),
                                   (20_011, 16, 1), (66_003, 64, 70)])
@pytest.mark.parametrize("shift", [0, 1, 4])
def test_update(kernel, N, M, K, shift):
    """shift: bytes by which the codes are moved off their alignment (1: read byte by byte)"""
    import torch

    import oracle
    import paper_1709_03708_amd as pq

    rng = np.random.default_rng(N + M)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    codes[: N // 2] = codes[0]                                   # a cluster whose codes are all alike
    a = rng.integers(-1, K + 1, N).astype(np.int32)              # some outside: not counted
    a[: N // 2] = 0
    t = rng.random((M, 256, 256), dtype=np.float32)
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    c = torch.from_numpy(centers.copy()).cuda()
    buf = torch.zeros(codes.size + shift, dtype=torch.uint8, device="cuda")
    x = buf[shift:].view(codes.shape)
    x.copy_(torch.from_numpy(codes))
    pq.set_option("hist_kernel", kernel)
    try:
        _, h, n = pq.update(x, torch.from_numpy(a).cuda(), torch.from_numpy(t).cuda(), c)
    finally:
        pq.set_option("hist_kernel", 0)
    valid = (a >= 0) & (a < K)
    rc, rh, rn = oracle.update(codes[valid], a[valid], t, centers)
    np.testing.assert_array_equal(u32(h), rh)
    np.testing.assert_array_equal(u32(n), rn)
    np.testing.assert_array_equal(c.cpu().numpy(), rc)


def test_large_fit_keeps_its_keys_or_knows_that_it_did_not():
    """M = 8 at a size where the lower-bound scan runs and the update now sorts: the keys' room is the sorted indices'."""
    import torch

    import paper_1709_03708_amd as pq

    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    N, M, K = 2_000_000, 8, 3600
    tmpl = torch.randint(0, 256, (K, M), generator=g, device="cuda", dtype=torch.uint8)
    x = tmpl[torch.randint(0, K, (N,), generator=g, device="cuda")]
    x = torch.where(torch.rand(N, M, generator=g, device="cuda") < 0.3,
                    torch.randint(0, 256, (N, M), generator=g, device="cuda", dtype=torch.uint8), x).contiguous()
    t = pq.build_tables(torch.randn(M, 256, 16, generator=g, device="cuda"))
    c0 = x[:K].contiguous()
    c1, c2 = c0.clone(), c0.clone()
    _, a1 = pq.fit(x, t, c1, 3)
    for _ in range(3):
        a2, _ = pq.assign(x, c2, t)
        pq.update(x, a2, t, c2)
    assert torch.equal(a1, a2) and torch.equal(c1, c2)
