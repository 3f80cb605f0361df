"""Histograms from indices sorted by cluster group: every block size of the scatter and its edges, groups of several sizes and a
ragged last one, heavy groups that several workgroups share, one cluster per group, and more groups than a block can count."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,K", [(2048, 8, 17), (2049, 8, 3001), (524_287, 4, 5000), (524_289, 12, 4001), (1_048_577, 6, 9001),
                                   (2_097_151, 8, 5000), (2_200_003, 4, 70_001), (4_194_305, 4, 3000), (300_007, 64, 300),
                                   (100_003, 64, 9000), (100_003, 64, 33_000), (60_001, 64, 1)])
@pytest.mark.parametrize("uneven", [False, True])
def test_histograms(N, M, K, uneven):
    import torch

    import oracle
    import paper_1709_03708_amd as pq

    g = torch.Generator(device="cuda")
    g.manual_seed(N + M)
    x = torch.randint(0, 256, (N, M), generator=g, device="cuda", dtype=torch.uint8)
    a = torch.randint(-1, K + 1, (N,), generator=g, device="cuda", dtype=torch.int32)     # some outside: not counted
    if uneven:
        a = torch.where(torch.rand(N, generator=g, device="cuda") < 0.6, torch.full_like(a, K // 2), a)
    t = torch.rand(M, 256, 256, generator=g, device="cuda")
    c = torch.randint(0, 256, (K, M), generator=g, device="cuda", dtype=torch.uint8)
    before = c.cpu().numpy()
    pq.set_option("hist_kernel", 3)
    try:
        _, h, n = pq.update(x, a, t, c)
    finally:
        pq.set_option("hist_kernel", 0)
    valid = (a >= 0) & (a < K)
    k, xv = a[valid].long(), x[valid]
    assert torch.equal(n.view(torch.int32).long(), torch.bincount(k, minlength=K))
    h = h.view(torch.int32).view(K, M, 256)
    for m in range(M):
        ref = torch.bincount(k * 256 + xv[:, m].long(), minlength=K * 256)
        assert torch.equal(h[:, m].reshape(-1).long(), ref)
    if K * M <= 300_000:                                                          # (their histograms: 300 MB on the host)
        want = oracle.vote(h.reshape(K, M, 256).cpu().numpy().view(np.uint32), n.cpu().numpy().view(np.uint32), t.cpu().numpy(), before)
        np.testing.assert_array_equal(c.cpu().numpy(), want)


# the smallest sizes at which the iterations of a fit sort by group, too few groups for the line that holds where scans keep their keys
@pytest.mark.parametrize("M,N,K", [(16, 100_000, 500), (16, 131_077, 641), (32, 100_003, 150), (32, 140_001, 399)])
@pytest.mark.parametrize("uneven", [False, True])
def test_fit(M, N, K, uneven):
    import torch

    import oracle
    import paper_1709_03708_amd as pq
    from _util import rand_tables

    assert pq.call_plan(N, M, K)["count"] == "sorted" and pq.call_plan(99_999, M, K)["count"] != "sorted"
    rng = np.random.default_rng(M + K)
    tables = rand_tables(rng, M)
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    of = rng.integers(0, K, N)
    if uneven:
        of[rng.random(N) < 0.6] = K // 2
    codes = centers[of]
    other = rng.random((N, M)) < 0.3
    codes[other] = rng.integers(0, 256, int(other.sum()), dtype=np.uint8)
    c = torch.from_numpy(centers).cuda()
    _, a = pq.fit(torch.from_numpy(codes).cuda(), torch.from_numpy(tables).cuda(), c, 2)
    want, ra, _, _ = oracle.fit(codes, tables, centers, 2)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(c.cpu().numpy(), want)
