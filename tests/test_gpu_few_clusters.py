"""The update with few clusters (one wave per cluster and subspace), and the scan on the matrix cores in front of the one with one lane
per center, against the oracle: edges of their launches and rules, uneven and empty clusters, tables that are not finite or no distances."""
from __future__ import annotations

import numpy as np
import pytest

from _util import rand_tables

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    import oracle
    import paper_1709_03708_amd as pq

    assert torch.cuda.is_available()
    return pq, oracle, torch


def _check_update(env, codes, assign, tables, K, offset=0):
    pq, oracle, torch = env
    N, M = codes.shape
    rng = np.random.default_rng(K)
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    buf = torch.empty(N * M + offset, dtype=torch.uint8, device="cuda")
    x = buf[offset:].view(N, M)
    x.copy_(torch.from_numpy(codes))
    c = torch.from_numpy(centers.copy()).cuda()
    _, h, n = pq.update(x, torch.from_numpy(assign).cuda(), torch.from_numpy(tables).cuda(), c)
    with np.errstate(all="ignore"):
        rc, rh, rn = oracle.update(codes, assign, tables, centers)
    np.testing.assert_array_equal(h.cpu().numpy().view(np.uint32), rh)
    np.testing.assert_array_equal(n.cpu().numpy().view(np.uint32), rn)
    np.testing.assert_array_equal(c.cpu().numpy(), rc)


# counted from the codes (up to 40000, 12000 byte by byte, K ceil(M / 4) <= compute units) and beyond, where partial histograms arrive
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (3, 12_000, 40), (3, 12_001, 40), (4, 10_240, 256), (4, 10_241, 257), (4, 40_000, 30), (4, 40_001, 30),
                                   (6, 700, 128), (8, 20_481, 128), (8, 9000, 129), (32, 5000, 32), (32, 5000, 33), (4, 400_000, 100),
                                   (8, 300_000, 60), (5, 150_000, 90), (16, 50_000, 40)])
@pytest.mark.parametrize("shape", ["even", "uneven", "one"])
def test_update(env, M, N, K, shape):
    rng = np.random.default_rng(M + N + K)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    codes[rng.random((N, M)) < 0.6] &= 15                                        # few and many non-zero bins
    if shape == "even":
        assign = rng.integers(0, K, N).astype(np.int32)
    elif shape == "uneven":
        assign = np.minimum(rng.random(N) ** 4 * K, K - 1).astype(np.int32)
    else:
        assign = np.full(N, K - 1, np.int32)                                     # all others are empty
    tables = rand_tables(rng, M)
    _check_update(env, codes, assign, tables, K, offset=N % 2)


@pytest.mark.parametrize("N,K", [(3000, 20), (100_000, 50)])
def test_update_with_ties_and_non_finite_tables(env, N, K):
    rng = np.random.default_rng(N)
    M = 4
    codes = rng.integers(0, 40, (N, M), dtype=np.uint8)
    assign = rng.integers(0, K, N).astype(np.int32)
    ham = np.ones((M, 256, 256), np.float32)
    ham[:, np.arange(256), np.arange(256)] = 0
    _check_update(env, codes, assign, ham, K)
    bad = rand_tables(rng, M)
    bad[rng.random(bad.shape) < 0.02] = np.nan
    bad[rng.random(bad.shape) < 0.02] = np.inf
    bad[1] = np.nan                                                              # no candidate can be taken
    bad[2, :, 7:] = np.inf
    _check_update(env, codes, assign, bad, K)


def _points(rng, M, dims):
    p = rng.standard_normal((M, 256, dims))
    return ((p[:, :, None, :] - p[:, None, :, :]) ** 2).sum(3).astype(np.float32)


# sizes on either side of the rule (128 and 256 dimensions in all), tables it is for and not for; the log has a scan more where it is tried
@pytest.mark.parametrize("M,N,K,tried", [(8, 36_001, 1000, True), (8, 20_000, 1000, False), (16, 24_000, 300, True), (16, 9000, 300, False),
                                         (16, 30_011, 1000, True), (32, 19_999, 300, True), (32, 5000, 160, False), (32, 11_003, 1500, True)])
@pytest.mark.parametrize("dims", [128, 256, 0])
def test_matrix_cores_before_one_lane_per_center(env, M, N, K, tried, dims):
    pq, oracle, torch = env
    rng = np.random.default_rng(N + K + dims)
    tables = _points(rng, M, dims // M) if dims else rand_tables(rng, M)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    centers = codes[rng.permutation(N)[:K]].copy()
    assert pq.scan_plan(N, M, K)["scan"] == 0
    d = [torch.from_numpy(v).cuda() for v in (codes, centers, tables)]
    pq.profile_read()
    pq.set_option("profile", 1)
    try:
        a, dist = pq.assign(*d)
    finally:
        pq.set_option("profile", 0)
    assert pq.profile_read()[1] == (2 if tried else 1)
    ra, rd = oracle.assign(codes, centers, tables)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(dist.cpu().numpy().view(np.uint32), rd.view(np.uint32))


@pytest.mark.parametrize("M", [8, 16])
@pytest.mark.parametrize("suited", [True, False])
def test_fit_with_both(env, M, suited):
    """Several iterations: the points are found once, the centers' fragments each time."""
    pq, oracle, torch = env
    rng = np.random.default_rng(M)
    N, K = 36_000, 1000
    tables = _points(rng, M, 128 // M) if suited else rand_tables(rng, M)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    centers = codes[:K].copy()
    c = torch.from_numpy(centers.copy()).cuda()
    _, a = pq.fit(torch.from_numpy(codes).cuda(), torch.from_numpy(tables).cuda(), c, 3)
    for _ in range(3):
        ra, _ = oracle.assign(codes, centers, tables)
        centers, _, _ = oracle.update(codes, ra, tables, centers)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(c.cpu().numpy(), centers)


@pytest.mark.parametrize("M,N,K", [(4, 2, 9000), (4, 1024, 513), (4, 1025, 513), (8, 3, 20_000), (8, 1025, 300), (32, 7, 3000), (16, 40, 64), (16, 40, 63)])
def test_rows_of_one_and_several_codes(env, M, N, K):
    """Codes per block, and centers split over blocks."""
    pq, oracle, torch = env
    rng = np.random.default_rng(N + K)
    codes = rng.integers(0, 20, (N, M), dtype=np.uint8)
    centers = rng.integers(0, 20, (K, M), dtype=np.uint8)
    tables = rand_tables(rng, M)
    a, dist = pq.assign(*[torch.from_numpy(v).cuda() for v in (codes, centers, tables)])
    ra, rd = oracle.assign(codes, centers, tables)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(dist.cpu().numpy().view(np.uint32), rd.view(np.uint32))
