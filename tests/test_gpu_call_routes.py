"""Calls at the edges of the rules that choose their scan or their count, against the oracle."""
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


def _off(torch, a, by):
    """a on the device, `by` bytes off its alignment"""
    buf = torch.empty(a.nbytes + by, dtype=torch.uint8, device="cuda")
    buf[by:].copy_(torch.from_numpy(a.view(np.uint8).reshape(-1)))
    return buf[by:].view(*a.shape)


def _check_assign(env, codes, centers, tables, centers_on=None):
    pq, oracle, torch = env
    x, t = torch.from_numpy(codes).cuda(), torch.from_numpy(tables).cuda()
    c = torch.from_numpy(centers).cuda() if centers_on is None else centers_on
    a, d = pq.assign(x, c, t)
    with np.errstate(all="ignore"):
        ra, rd = oracle.assign(codes, centers, tables)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), rd.view(np.uint32))


@pytest.mark.parametrize("M,N,K", [(4, 19_459, 300), (4, 19_460, 300), (8, 19_460, 300), (16, 19_460, 300), (32, 19_460, 300)])
def test_centers_off_their_alignment(env, M, N, K):
    rng = np.random.default_rng(N + M)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    centers = codes[rng.permutation(N)[:K]].copy()
    _check_assign(env, codes, centers, rand_tables(rng, M), _off(env[2], centers, 1 + M % 3))


# one lane per center: two codes per block (M = 4, 16), parts of the centers, a ragged last code and part, rows in LDS or not
@pytest.mark.parametrize("M,N,K", [(4, 300, 1000), (4, 2101, 1000), (4, 1025, 20_001), (4, 257, 60_003), (8, 257, 30_000), (16, 2101, 513), (16, 1501, 2500),
                                   (16, 1025, 9001), (32, 257, 9000), (32, 3, 5000), (16, 300, 95), (16, 300, 96)])
@pytest.mark.parametrize("ties", [False, True])
def test_rows_and_parts(env, M, N, K, ties):
    rng = np.random.default_rng(N + K)
    top = 8 if ties else 256
    codes, centers = rng.integers(0, top, (N, M), dtype=np.uint8), rng.integers(0, top, (K, M), dtype=np.uint8)
    tables = rand_tables(rng, M, integer=ties)
    if ties:
        tables[0, 3] = np.inf
        tables[M - 1, 5] = np.nan                                                # codes without any distance
    _check_assign(env, codes, centers, tables)


@pytest.mark.parametrize("M,N,K", [(8, 36_001, 1000), (16, 30_011, 1000), (32, 11_003, 1500)])
@pytest.mark.parametrize("blocks", [1, 3, 1000])
def test_single_codes_left_by_the_matrix_cores(env, M, N, K, blocks):
    """Stretches of codes that are as far from 200 centers, no two of them equal: few of them are left to one lane per center, and no
    others; all of them, and everything is.  The scan's state is the end of the workspace: word 0 is for everything, word 12 for some."""
    pq, oracle, torch = env
    rng = np.random.default_rng(M + blocks)
    cw = rng.standard_normal((M, 256, 128 // M)).astype(np.float32)
    cw[M - 1, :200] = cw[M - 1, 0]
    tables = oracle.build_tables(cw)
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    order = rng.permutation(K)
    alike, others = order[:200], order[200:]
    centers[alike] = centers[alike[0]]
    centers[alike, M - 1] = np.arange(200)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    near = rng.random((N, M)) < 0.8
    codes[near] = centers[others[rng.integers(0, K - 200, N)]][near]
    for b in range(min(blocks, N // 2048)):
        codes[b * 2048 + 100: b * 2048 + 500 if blocks < 1000 else N] = centers[alike[7]]
    ws = torch.full((pq.workspace_bytes(N, M, K),), 0xA5, dtype=torch.uint8, device="cuda")
    assert pq.call_plan(N, M, K, dist=True)["dot"]
    a, d = pq.assign(*[torch.from_numpy(v).cuda() for v in (codes, centers, tables)], workspace=ws)
    state = ws[-256:].view(torch.int32).cpu().numpy()
    ra, rd = oracle.assign(codes, centers, tables)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), rd.view(np.uint32))
    assert (state[0] == 0 and state[12] == 1) if blocks < 1000 else state[0] == 1
    c = torch.from_numpy(centers).cuda()
    _, a = pq.fit(torch.from_numpy(codes).cuda(), torch.from_numpy(tables).cuda(), c, 2)
    want = centers
    for _ in range(2):
        ra, _ = oracle.assign(codes, want, tables)
        want, _, _ = oracle.update(codes, ra, tables, want)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(c.cpu().numpy(), want)


# the vote counts: one, two and four subspaces per workgroup, read as words and byte by byte, and what lies beyond its limits
@pytest.mark.parametrize("M,N,K", [(4, 40_000, 64), (4, 30_001, 65), (4, 10_241, 129), (4, 10_240, 256), (8, 511, 32), (8, 20_481, 64), (3, 12_000, 85), (3, 12_000, 86),
                                   (6, 12_000, 43), (6, 1499, 128), (1, 9, 1), (4, 28_001, 8), (64, 10_241, 16)])
@pytest.mark.parametrize("codes_are", ["spread", "alike", "two", "one word"])
def test_vote_counts_heavy_clusters(env, M, N, K, codes_are):
    pq, oracle, torch = env
    rng = np.random.default_rng(N + K)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    assign = rng.integers(-1, K + 1, N).astype(np.int32)                         # some outside: not counted
    if codes_are != "spread":
        assign[N // 5:] = K - 1
        codes[:] = codes[0] if codes_are == "alike" else codes[rng.integers(0, 2, N)] if codes_are == "two" else codes[:, :1]
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    tables = rand_tables(rng, M)
    c = torch.from_numpy(centers.copy()).cuda()
    _, h, n = pq.update(torch.from_numpy(codes).cuda(), torch.from_numpy(assign).cuda(), torch.from_numpy(tables).cuda(), c)
    inside = (assign >= 0) & (assign < K)
    rc, rh, rn = oracle.update(codes[inside], assign[inside], tables, centers)
    np.testing.assert_array_equal(h.cpu().numpy().view(np.uint32), rh)
    np.testing.assert_array_equal(n.cpu().numpy().view(np.uint32), rn)
    np.testing.assert_array_equal(c.cpu().numpy(), rc)


# histograms by subspace from their smallest sizes on, codes off their alignment
@pytest.mark.parametrize("M,N,K", [(4, 1_000_000, 33), (5, 1_500_000, 32), (4, 1_000_003, 100), (7, 1_000_001, 48), (16, 2_200_001, 64), (8, 1_700_000, 100)])
@pytest.mark.parametrize("off", [0, 1])
def test_histograms_by_subspace(env, M, N, K, off):
    pq, oracle, torch = env
    rng = np.random.default_rng(N + M)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    codes[:, 0] &= 3                                                             # many members in few bins
    assign = rng.integers(0, K, N).astype(np.int32)
    assign[: N // 2] = K - 1
    centers, tables = rng.integers(0, 256, (K, M), dtype=np.uint8), rand_tables(rng, M)
    assert pq.call_plan(N, M, K, codes_aligned=not off)["count"] == "subspaces"
    c = torch.from_numpy(centers.copy()).cuda()
    _, h, n = pq.update(_off(torch, codes, off), torch.from_numpy(assign).cuda(), torch.from_numpy(tables).cuda(), c)
    rc, rh, rn = oracle.update(codes, assign, tables, centers)
    np.testing.assert_array_equal(h.cpu().numpy().view(np.uint32), rh)
    np.testing.assert_array_equal(n.cpu().numpy().view(np.uint32), rn)
    np.testing.assert_array_equal(c.cpu().numpy(), rc)


# the owner path's adds: chunks of four words and what is left over, its queue full (nearly all codes in one group), codes byte by byte
@pytest.mark.parametrize("M,N,K", [(4, 150_000, 3), (8, 150_000, 2), (12, 100_003, 5), (16, 100_000, 17), (20, 150_001, 2), (28, 70_000, 9), (40, 60_000, 130), (64, 50_000, 2), (5, 100_000, 7)])
def test_owner_histograms_of_heavy_clusters(env, M, N, K):
    pq, oracle, torch = env
    rng = np.random.default_rng(N + M)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    assign = np.where(rng.random(N) < 0.9, K - 1, rng.integers(-1, K + 1, N)).astype(np.int32)
    centers, tables = rng.integers(0, 256, (K, M), dtype=np.uint8), rand_tables(rng, M)
    c = torch.from_numpy(centers.copy()).cuda()
    pq.set_option("hist_kernel", 2)
    try:
        assert pq.call_plan(N, M, K)["count"] == "cluster_groups"
        _, h, n = pq.update(torch.from_numpy(codes).cuda(), torch.from_numpy(assign).cuda(), torch.from_numpy(tables).cuda(), c)
    finally:
        pq.set_option("hist_kernel", 0)
    inside = (assign >= 0) & (assign < K)
    rc, rh, rn = oracle.update(codes[inside], assign[inside], tables, centers)
    np.testing.assert_array_equal(h.cpu().numpy().view(np.uint32), rh)
    np.testing.assert_array_equal(n.cpu().numpy().view(np.uint32), rn)
    np.testing.assert_array_equal(c.cpu().numpy(), rc)


# the vote with a workgroup per cluster: grids that the eight dies do not divide, more subspaces than clusters and the other way round
@pytest.mark.parametrize("M,N,K", [(1, 50_000, 1), (4, 50_000, 9), (5, 50_000, 3), (20, 46_000, 8), (24, 46_000, 4), (40, 41_000, 28), (40, 41_000, 1), (60, 41_000, 17), (12, 60_000, 3)])
def test_vote_per_cluster_by_dies(env, M, N, K):
    pq, oracle, torch = env
    rng = np.random.default_rng(N + M)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    assign = rng.integers(0, K, N).astype(np.int32)
    centers, tables = rng.integers(0, 256, (K, M), dtype=np.uint8), rand_tables(rng, M)
    assert pq.call_plan(N, M, K)["vote_per_cluster"]
    c = torch.from_numpy(centers.copy()).cuda()
    _, h, n = pq.update(torch.from_numpy(codes).cuda(), torch.from_numpy(assign).cuda(), torch.from_numpy(tables).cuda(), c)
    rc, rh, rn = oracle.update(codes, assign, tables, centers)
    np.testing.assert_array_equal(h.cpu().numpy().view(np.uint32), rh)
    np.testing.assert_array_equal(n.cpu().numpy().view(np.uint32), rn)
    np.testing.assert_array_equal(c.cpu().numpy(), rc)
