"""The update with few clusters (one wave per cluster and subspace) against the oracle: edges of its launches and rules, uneven and
empty clusters, tables that are not finite."""
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
