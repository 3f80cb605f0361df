"""The update step on clusters of very uneven size and on few clusters, against the oracle: shared groups of the sorted
histogram, block-wise scatter, the histogram by subspace, dropped assignments."""
from __future__ import annotations

import numpy as np
import pytest

from _util import rand_tables, u32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    import oracle
    import paper_1709_03708_amd as pq

    assert torch.cuda.is_available()
    return pq, oracle, torch


def _assignment(rng, kind, N, K):
    if kind == "even":
        return rng.integers(0, K, N)
    if kind == "one":
        return np.full(N, K - 1)
    if kind == "heavy":
        return np.where(rng.random(N) < 0.7, K // 2, rng.integers(0, K, N))
    return np.minimum((rng.pareto(0.7, N) * 2).astype(np.int64), K - 1)           # "tail"


@pytest.mark.parametrize("M,N,K,hist_kernel", [
    (4, 90_001, 1, 0), (4, 70_003, 100, 0), (4, 70_001, 128, 0), (4, 9001, 129, 0), (8, 70_000, 31, 0), (3, 70_007, 60, 0),
    (16, 66_001, 128, 0), (32, 65_536, 17, 0), (6, 66_000, 33, 0), (8, 60_001, 500, 3), (8, 200_003, 3000, 3), (4, 30_000, 9000, 3),
    (32, 30_001, 300, 3), (5, 40_000, 700, 3), (4, 20_000, 33_000, 3),
    # shares of heavy groups, few and many of them, and as many groups as codes would fill
    (4, 400_000, 33, 3), (4, 300_000, 9000, 3), (32, 150_000, 2000, 3), (64, 40_000, 130, 3), (4, 500_000, 30_000, 0),
    # counted by subspace: all clusters of one or several subspaces in a workgroup
    (4, 1_200_001, 33, 0), (4, 1_200_003, 100, 0), (4, 1_200_007, 128, 0), (6, 1_800_001, 61, 0), (8, 2_400_000, 100, 0),
    (16, 1_000_009, 17, 0), (32, 1_000_001, 31, 0)])
@pytest.mark.parametrize("kind", ["even", "one", "heavy", "tail"])
def test_update(env, M, N, K, hist_kernel, kind):
    pq, oracle, torch = env
    rng = np.random.default_rng(N + K + M)
    codes = np.where(rng.random((N, M)) < 0.5, 7, rng.integers(0, 256, (N, M))).astype(np.uint8)
    a = _assignment(rng, kind, N, K).astype(np.int32)
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    tables = rand_tables(rng, M)
    d = torch.from_numpy(centers).cuda()
    pq.set_option("hist_kernel", hist_kernel)
    try:
        _, h, c = pq.update(torch.from_numpy(codes).cuda(), torch.from_numpy(a).cuda(), torch.from_numpy(tables).cuda(), d)
    finally:
        pq.set_option("hist_kernel", 0)
    rcen, rh, rc = oracle.update(codes, a, tables, centers)
    np.testing.assert_array_equal(u32(h), rh)
    np.testing.assert_array_equal(u32(c), rc)
    np.testing.assert_array_equal(d.cpu().numpy(), rcen)


@pytest.mark.parametrize("N,K,hist_kernel", [(70_001, 100, 0), (1_200_001, 100, 0), (70_001, 2000, 3)])
def test_dropped_assignments(env, N, K, hist_kernel):
    """Values outside [0, K) are ignored."""
    pq, oracle, torch = env
    rng = np.random.default_rng(K)
    M = 4
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    a = rng.integers(-3, K + 3, N).astype(np.int32)
    a[:5] = [-2**31, 2**31 - 1, K, -1, K + 1]
    tables = rand_tables(rng, M)
    d = torch.zeros((K, M), dtype=torch.uint8, device="cuda")
    pq.set_option("hist_kernel", hist_kernel)
    try:
        _, h, c = pq.update(torch.from_numpy(codes).cuda(), torch.from_numpy(a).cuda(), torch.from_numpy(tables).cuda(), d)
    finally:
        pq.set_option("hist_kernel", 0)
    ok = (a >= 0) & (a < K)
    _, rh, rc = oracle.update(codes[ok], a[ok], tables, np.zeros((K, M), np.uint8))
    np.testing.assert_array_equal(u32(h), rh)
    np.testing.assert_array_equal(u32(c), rc)
