"""The scan with one lane per center against the oracle: edges of its blocks and splits, every operand width, misaligned
operands, ties, non-finite tables."""
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


def _moved(torch, x, offset):
    buf = torch.empty(x.size + offset, dtype=getattr(torch, str(x.dtype)), device="cuda")
    v = buf[offset:].view(x.shape)
    v.copy_(torch.from_numpy(x))
    return v


def _check(env, codes, centers, tables, forced, offset=0):
    pq, oracle, torch = env
    N = codes.shape[0]
    a = torch.full((N,), -7, dtype=torch.int32, device="cuda")
    d = torch.full((N,), float("nan"), dtype=torch.float32, device="cuda")
    pq.set_option("assign_kernel", 1 if forced else 0)
    try:
        pq.assign(_moved(torch, codes, offset), _moved(torch, centers, offset), _moved(torch, tables, offset), assign=a, dist=d)
    finally:
        pq.set_option("assign_kernel", 0)
    with np.errstate(all="ignore"):
        ra, rd = oracle.assign(codes, centers, tables)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), rd.view(np.uint32))


@pytest.mark.parametrize("M", [1, 3, 4, 8, 12, 16, 32, 64])
@pytest.mark.parametrize("N,K", [(1, 1), (1, 159), (3, 160), (9, 255), (17, 257), (48, 1000), (1, 5003), (2049, 130), (4097, 513)])
def test_edges(env, M, N, K):
    rng = np.random.default_rng(M * 7 + N + K)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    tables = rand_tables(rng, M)
    _check(env, codes, centers, tables, forced=True)
    _check(env, codes, centers, tables, forced=False, offset=N % 3)


@pytest.mark.parametrize("M", [4, 8, 32, 6])
@pytest.mark.parametrize("K", [100, 600])
def test_ties_and_non_finite(env, M, K):
    rng = np.random.default_rng(M + K)
    codes = rng.integers(0, 30, (700, M), dtype=np.uint8)
    centers = rng.integers(0, 30, (K, M), dtype=np.uint8)
    ham = np.ones((M, 256, 256), np.float32)
    ham[:, np.arange(256), np.arange(256)] = 0
    _check(env, codes, centers, ham, forced=False)
    bad = rand_tables(rng, M)
    bad[rng.random(bad.shape) < 0.05] = np.nan
    bad[rng.random(bad.shape) < 0.05] = np.inf
    bad[rng.random(bad.shape) < 0.002] = -np.inf
    _check(env, codes, centers, bad, forced=False)
    bad[0] = np.nan
    _check(env, codes, centers, bad, forced=False)
