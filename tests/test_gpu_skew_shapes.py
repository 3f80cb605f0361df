"""The M = 4 skewed scan in the shapes of 2560 and 3072 codes per workgroup against the oracle: edges of workgroups, tiles and rounds, ties,
entries that are not finite, and where the default takes them."""
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


def _check(env, codes, centers, tables, variant):
    pq, oracle, torch = env
    pq.set_option("scan_variant", variant)
    try:
        a, d = pq.assign(*[torch.from_numpy(v).cuda() for v in (codes, centers, tables)])
    finally:
        pq.set_option("scan_variant", 0)
    with np.errstate(all="ignore"):
        ra, rd = oracle.assign(codes, centers, tables)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), rd.view(np.uint32))


@pytest.mark.parametrize("variant,C", [(38, 2560), (39, 3072)])
@pytest.mark.parametrize("K", [1, 32, 33, 100])
def test_edges(env, variant, C, K):
    rng = np.random.default_rng(K)
    for N in (1, C - 1, C, C + 1, 3 * C + 7):
        codes = rng.integers(0, 256, (N, 4), dtype=np.uint8)
        _check(env, codes, rng.integers(0, 256, (K, 4), dtype=np.uint8), rand_tables(rng, 4), variant)
    ham = np.ones((4, 256, 256), np.float32)
    ham[:, np.arange(256), np.arange(256)] = 0
    codes, centers = rng.integers(0, 20, (2 * C, 4), dtype=np.uint8), rng.integers(0, 20, (K, 4), dtype=np.uint8)
    _check(env, codes, centers, ham, variant)
    bad = rand_tables(rng, 4)
    bad[rng.random(bad.shape) < 0.05] = np.nan
    bad[rng.random(bad.shape) < 0.05] = np.inf
    bad[rng.random(bad.shape) < 0.002] = -np.inf
    _check(env, codes, centers, bad, variant)


# the default: 2560 codes, 3072, 4096, 2048, one assignment with more than 128 centers, and M = 8 in rounds of 1536
@pytest.mark.parametrize("M,N,K,variant", [(4, 655_360, 64, 38), (4, 786_000, 40, 39), (4, 786_433, 100, 34), (4, 1_000_000, 32, 37),
                                           (4, 600_001, 300, 38), (8, 530_001, 60, 2)])
def test_default(env, M, N, K, variant):
    pq, _, torch = env
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert pq.call_plan(N, M, K)["variant"] == variant
    rng = np.random.default_rng(N)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    _check(env, codes, codes[:K].copy(), rand_tables(rng, M), 0)
