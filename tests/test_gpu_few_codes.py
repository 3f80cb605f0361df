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


@pytest.mark.parametrize("M,N,K", [(1, 20_000, 1), (1, 20_000, 59), (3, 100_000, 60), (6, 100_000, 45), (6, 100_000, 46), (24, 20_000, 4),
                                   (24, 30_011, 12), (64, 20_000, 2), (12, 3000, 300), (6, 3000, 1249), (6, 3000, 1251)])
def test_few_centers(env, M, N, K):
    """Both sides of the limits between one lane per code and one per center, with and without the rows in LDS."""
    rng = np.random.default_rng(M + N + K)
    codes = rng.integers(0, 40, (N, M), dtype=np.uint8)
    centers = rng.integers(0, 40, (K, M), dtype=np.uint8)
    _check(env, codes, centers, rand_tables(rng, M), forced=False)
    if N >= 20_000:
        four = rng.integers(0, 256, (N, 4), dtype=np.uint8)                      # misaligned codes
        _check(env, four, rng.integers(0, 256, (min(K, 50), 4), dtype=np.uint8), rand_tables(rng, 4), forced=False, offset=1)


@pytest.mark.parametrize("M,K", [(1, 4), (6, 4), (24, 1)])
def test_few_centers_take_no_block_per_code(env, M, K):
    """400000 codes against a handful of centers: 10 to 50 times the time with a workgroup for every code."""
    pq, _, torch = env
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    N = 400_000
    codes = torch.randint(0, 256, (N, M), generator=g, device="cuda", dtype=torch.uint8)
    tables = torch.rand(M, 256, 256, generator=g, device="cuda")
    ws = torch.empty(pq.workspace_bytes(N, M, K), dtype=torch.uint8, device="cuda")
    a = torch.empty(N, dtype=torch.int32, device="cuda")

    def best_us():
        times = []
        for _ in range(5):
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s.record()
            pq.assign(codes, codes[:K].contiguous(), tables, assign=a, workspace=ws)
            e.record()
            torch.cuda.synchronize()
            times.append(s.elapsed_time(e) * 1e3)
        return min(times)

    assert best_us() < 200.0                                                     # 30 to 70 us against 310 to 940


@pytest.mark.parametrize("M,N,K", [(4, 10_000, 100), (4, 48, 1000), (6, 100_000, 3), (6, 5000, 2000), (4, 100_000, 100)])
def test_scan_event_log_has_every_scan(env, M, N, K):
    """Bit 0 of "profile" brackets the scan of any call, whichever it is."""
    pq, _, torch = env
    codes = torch.zeros(N, M, dtype=torch.uint8, device="cuda")
    tables = torch.rand(M, 256, 256, device="cuda")
    pq.profile_read()
    pq.set_option("profile", 1)
    try:
        for _ in range(3):
            pq.assign(codes, torch.zeros(K, M, dtype=torch.uint8, device="cuda"), tables)
    finally:
        pq.set_option("profile", 0)
    ms, launches = pq.profile_read()
    assert launches == 3 and ms > 0.0
