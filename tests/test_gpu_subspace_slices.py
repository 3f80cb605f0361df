"""Histograms of few clusters from slices of the codes: 16-bit counters up to their limit (a slice of equal codes in one cluster),
32-bit ones beyond, ragged slices, one and several subspaces per workgroup, unaligned codes."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,K", [(1_200_000, 4, 32), (1_281_167, 4, 100), (2_400_001, 8, 128), (1_000_000, 16, 31), (1_000_003, 64, 5),
                                   (4_100_000, 4, 64), (4_128_768, 4, 40), (4_128_769, 4, 40), (4_800_003, 16, 33)])
@pytest.mark.parametrize("alike", [False, True])
@pytest.mark.parametrize("shift", [0, 1])
def test_histograms(N, M, K, alike, shift):
    import torch

    import paper_1709_03708_amd as pq

    g = torch.Generator(device="cuda")
    g.manual_seed(N + M)
    buf = torch.randint(0, 256, (N * M + shift,), generator=g, device="cuda", dtype=torch.uint8)
    x = buf[shift:].view(N, M)
    a = torch.randint(-1, K + 1, (N,), generator=g, device="cuda", dtype=torch.int32)      # some outside: not counted
    if alike:
        x[: N - 1000] = x[0].clone()
        a[: N - 1000] = K - 1
    t = torch.rand(M, 256, 256, generator=g, device="cuda")
    c0 = torch.randint(0, 256, (K, M), generator=g, device="cuda", dtype=torch.uint8)
    c = c0.clone()
    _, h, n = pq.update(x, a, t, c)
    valid = (a >= 0) & (a < K)
    k, xv = a[valid].long(), x[valid]
    assert torch.equal(n.view(torch.int32).long(), torch.bincount(k, minlength=K))
    h = h.view(torch.int32).view(K, M, 256)
    for m in range(M):
        ref = torch.bincount(k * 256 + xv[:, m].long(), minlength=K * 256)
        assert torch.equal(h[:, m].reshape(-1).long(), ref)
    other = c0.clone()
    pq.set_option("hist_kernel", 3)
    try:
        pq.update(x, a, t, other)
    finally:
        pq.set_option("hist_kernel", 0)
    assert torch.equal(c, other)
