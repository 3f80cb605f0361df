"""The scan on the matrix cores against the oracle, where it can go wrong: edges of tiles, chunks and blocks, both numbers of
dimensions, tables that no points describe (which it must leave to the scans behind), ties and repeated centers, sums whose
order is the definition's.  All results are compared bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from _util import rand_tables, u32

pytestmark = pytest.mark.gpu

FORCED = 20


@pytest.fixture(scope="module")
def env():
    import torch

    import oracle
    import paper_1709_03708_amd as pq

    assert torch.cuda.is_available()
    yield pq, oracle, torch
    pq.set_option("scan_variant", 0)


def _problem(rng, N, M, K, Ds, spread=1.0):
    """Codes of clustered data (half of the subcodes of a template), tables of random codewords; some centers repeat."""
    cw = (rng.standard_normal((M, 256, Ds)) * spread).astype(np.float32)
    tmpl = rng.integers(0, 256, (max(K // 2, 1), M), dtype=np.uint8)
    codes = tmpl[rng.integers(0, tmpl.shape[0], N)]
    codes = np.where(rng.random((N, M)) < 0.3, rng.integers(0, 256, (N, M), dtype=np.uint8), codes)
    centers = codes[rng.integers(0, N, K)].copy()
    return cw, np.ascontiguousarray(codes), np.ascontiguousarray(centers)


def _check(env, codes, centers, tables, offset=0, dist=True, shift=0, left=None, variant=FORCED):
    """offset: floats by which the tables are moved off their alignment, shift: bytes likewise for codes and centers; left: whether
    the scan on the matrix cores, which has to be tried, hands the codes to the scans behind it"""
    pq, oracle, torch = env
    (N, M), K = codes.shape, centers.shape[0]

    def moved(v):
        buf = torch.zeros(v.size + shift, dtype=torch.uint8, device="cuda")
        buf[shift:] = torch.from_numpy(v.reshape(-1)).cuda()
        return buf[shift:].view(v.shape)

    buf = torch.empty(tables.size + offset, dtype=torch.float32, device="cuda")
    t = buf[offset:].view(tables.shape)
    t.copy_(torch.from_numpy(tables))
    a = torch.full((N,), -7, dtype=torch.int32, device="cuda")
    d = torch.full((N,), float("nan"), dtype=torch.float32, device="cuda") if dist else None
    ws = torch.full((pq.workspace_bytes(N, M, K),), 0xA5, dtype=torch.uint8, device="cuda")
    pq.set_option("scan_variant", variant)
    try:
        pq.assign(moved(codes), moved(centers), t, assign=a, dist=d, want_dist=dist, workspace=ws)
        if left is not None:
            assert pq.dot_scan(N, M, K, ws) == dict(tried=True, left=left)
    finally:
        pq.set_option("scan_variant", 0)
    ra, rd = oracle.assign(codes, centers, tables)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    if dist:
        np.testing.assert_array_equal(d.cpu().numpy(), rd)


# M = 4 keeps its own scans
LEFT_TO_OTHERS = {4: None, 8: False, 16: False, 32: False}


# with these the images leave room for the scan (M = 8: from 17 centers on)
MIN_K = {4: 128, 8: 64, 16: 32, 32: 33}


@pytest.mark.parametrize("M", [4, 8, 16, 32])
@pytest.mark.parametrize("N,dK", [(1, 0), (31, 1), (257, 31), (511, 32), (513, 33), (70001, 100)])
@pytest.mark.parametrize("dims", [96, 128, 256])
def test_sizes(env, M, N, dK, dims):
    pq, oracle, _ = env
    rng = np.random.default_rng(1000 * M + N + dims)
    cw, codes, centers = _problem(rng, N, M, MIN_K[M] + dK, dims // M)
    _check(env, codes, centers, oracle.build_tables(cw), offset=N % 3, dist=N != 511, left=LEFT_TO_OTHERS[M])


@pytest.mark.parametrize("M", [4, 8, 16, 32])
@pytest.mark.parametrize("shift", [4, 8, 12, 1])
def test_operands_off_their_alignment(env, M, shift):
    """Codes and centers are read as words (shift 1: left to the scans that read bytes)."""
    pq, oracle, _ = env
    rng = np.random.default_rng(M + shift)
    cw, codes, centers = _problem(rng, 1501, M, 133, 128 // M)
    _check(env, codes, centers, oracle.build_tables(cw), shift=shift)


@pytest.mark.parametrize("M", [8, 32])
def test_many_centers_and_blocks(env, M):
    """Several chunks of centers, several blocks of codes per workgroup."""
    pq, oracle, _ = env
    rng = np.random.default_rng(M)
    cw, codes, centers = _problem(rng, 300_001, M, 333, 128 // M)
    _check(env, codes, centers, oracle.build_tables(cw), dist=False, left=False)


@pytest.mark.parametrize("M", [4, 8, 16, 32])
@pytest.mark.parametrize("kind", ["random", "integer", "hamming", "lattice", "constant", "nan", "inf", "huge", "tiny", "negative",
                                  "wide"])
def test_tables(env, M, kind):
    """Tables that no few points describe, that tie everywhere, or that the halves cannot hold."""
    pq, oracle, _ = env
    rng = np.random.default_rng(M)
    cw, codes, centers = _problem(rng, 3001, M, 150, 128 // M)
    t = oracle.build_tables(cw)
    i = np.arange(256)
    if kind == "random":
        t = rand_tables(rng, M)
    elif kind == "integer":
        t = rand_tables(rng, M, integer=True)
    elif kind == "hamming":
        t = np.unpackbits((i[:, None] ^ i).astype(np.uint8)[..., None], axis=-1).sum(-1).astype(np.float32)
        t = np.ascontiguousarray(np.broadcast_to(t, (M, 256, 256)))
    elif kind == "lattice":
        t = np.ascontiguousarray(np.broadcast_to(((i[:, None] - i) ** 2).astype(np.float32), (M, 256, 256)))
    elif kind == "constant":
        t = np.ones((M, 256, 256), np.float32)
    elif kind == "nan":
        t[M // 2, 3, 5] = np.nan
    elif kind == "inf":
        t[0, 7, 9] = np.inf
        t[M - 1, 0, 0] = -np.inf
    elif kind == "huge":
        t = (t * np.float32(1e30)).astype(np.float32)
    elif kind == "tiny":
        t = (t * np.float32(1e-30)).astype(np.float32)
    elif kind == "negative":
        t = t - np.float32(3.0)                    # a constant that all distances share, but not on the diagonal of any points
    elif kind == "wide":
        t = oracle.build_tables(rng.standard_normal((M, 256, 300 // M + 1)).astype(np.float32))
    kept = kind in ("lattice", "huge", "tiny") or (kind == "hamming" and M == 32)
    _check(env, codes, centers, t, dist=kind != "integer", left=None if M == 4 else not kept)


@pytest.mark.parametrize("M", [8, 16, 32])
@pytest.mark.parametrize("kind", ["sample spans half", "sample is one point", "too many outside the sample", "repeated", "scales",
                                  "one subspace", "ranks"])
def test_points(env, M, kind):
    """Codewords 0..15, 64..79, 128..143, 192..207 are factorised first; what they do not span is found afterwards."""
    pq, oracle, _ = env
    rng = np.random.default_rng(M + len(kind))
    r = 256 // M
    first = np.arange(256) % 64 < 16
    cw, codes, centers = _problem(rng, 2003, M, 140, r + 1 if kind.startswith("too many") else r)
    if kind == "sample spans half":
        cw[:, first, r // 2:] = 0.0
    elif kind == "sample is one point":
        cw[:, first] = cw[:, :1]
    elif kind == "too many outside the sample":
        cw[:, first, r // 2:] = 0.0
    elif kind == "repeated":
        cw[:, 40:] = cw[:, :216] + 0.0
        cw[:, 200:] = cw[:, 3:4]
    elif kind == "scales":
        cw *= (np.float32(2.0) ** (np.arange(M) % 5 - 2).astype(np.float32))[:, None, None]
    elif kind == "one subspace":
        cw[1:] = 0.0
    elif kind == "ranks":
        for m in range(M):
            cw[m, :, 1 + m % r:] = 0.0
    _check(env, codes, centers, oracle.build_tables(cw), left=None if kind == "one subspace" else kind.startswith("too many"))


@pytest.mark.parametrize("M", [8, 16, 32])
@pytest.mark.parametrize("levels,left", [(2, True), (9, False)])
def test_tables_of_few_values(env, M, levels, left):
    """Codewords on a grid: left where the distances take few values in all subspaces, not where one subspace takes many."""
    pq, oracle, _ = env
    rng = np.random.default_rng(M + levels)
    cw, codes, centers = _problem(rng, 2001, M, 150, 128 // M)
    cw[:] = np.float32(0.3) * rng.integers(0, levels, cw.shape)
    if left:
        cw[:, :, 2:] = 0.0
        _check(env, codes, centers, oracle.build_tables(cw), left=True)
        cw[0] = rng.standard_normal(cw[0].shape)
        _check(env, codes, centers, oracle.build_tables(cw))
    else:
        _check(env, codes, centers, oracle.build_tables(cw), left=False)


@pytest.mark.parametrize("M", [8, 16, 32])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_one_entry_that_is_not_finite(env, M, value):
    """Off the first row and the diagonal, and so few codes and centers that giving all their distances exceeds none of the scan's own
    limits: it is the check of the tables that leaves them."""
    pq, oracle, _ = env
    rng = np.random.default_rng(M)
    cw, codes, centers = _problem(rng, 3, M, 66, 128 // M)
    for at in ((0, 7, 9), (M - 1, 250, 3), (M // 2, 255, 254)):
        t = oracle.build_tables(cw)
        t[at] = value
        _check(env, codes, centers, t, left=True)


@pytest.mark.parametrize("M", [8, 16])
def test_near_ties_are_decided_by_the_sum_of_the_definition(env, M):
    """Codewords on few values: thousands of centers at distances that differ in the last bits or not at all."""
    pq, oracle, _ = env
    rng = np.random.default_rng(3 * M)
    cw, codes, centers = _problem(rng, 4001, M, 700, 128 // M)
    cw = np.round(cw * 2.0).astype(np.float32) * np.float32(0.1)
    _check(env, codes, centers, oracle.build_tables(cw), left=False)
    one = np.repeat(centers[:1], 64, axis=0)       # one center, 64 times
    _check(env, codes, np.ascontiguousarray(one), oracle.build_tables(cw))


@pytest.mark.parametrize("M,N,K", [(8, 40_003, 200), (16, 30_001, 320), (32, 20_001, 450)])
def test_fit(env, M, N, K):
    """Iterations of one call: the points are found once, the centers move."""
    pq, oracle, torch = env
    rng = np.random.default_rng(M + N)
    cw, codes, centers = _problem(rng, N, M, K, 128 // M)
    t = oracle.build_tables(cw)
    c = torch.from_numpy(centers).cuda()
    h = torch.empty((K, M, 256), dtype=torch.int32, device="cuda")
    n = torch.empty(K, dtype=torch.int32, device="cuda")
    ws = torch.full((pq.workspace_bytes(N, M, K),), 0xA5, dtype=torch.uint8, device="cuda")
    pq.set_option("scan_variant", FORCED)
    try:
        _, a = pq.fit(torch.from_numpy(codes).cuda(), torch.from_numpy(t).cuda(), c, 4, hist=h, counts=n, workspace=ws)
        assert pq.dot_scan(N, M, K, ws) == dict(tried=True, left=False)
    finally:
        pq.set_option("scan_variant", 0)
    want = centers
    for _ in range(4):
        ra, _ = oracle.assign(codes, want, t)
        want, rh, rn = oracle.update(codes, ra, t, want)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(c.cpu().numpy(), want)
    np.testing.assert_array_equal(u32(h), rh)
    np.testing.assert_array_equal(u32(n), rn)


def _alike(rng, N, M, K, same):
    """Codewords of the last subspace that are all one point, and centers in groups of `same` that differ there only: every code is
    as far from all of a group, though no center repeats another.  The tables are those of points all the same."""
    cw = rng.standard_normal((M, 256, 128 // M)).astype(np.float32)
    cw[M - 1] = cw[M - 1, :1]
    centers = np.repeat(rng.integers(0, 256, ((K + same - 1) // same, M), dtype=np.uint8), same, axis=0)[:K]
    centers[:, M - 1] = np.arange(K) % same
    codes = centers[rng.integers(0, K, N)]
    codes = np.where(rng.random((N, M)) < 0.2, rng.integers(0, 256, (N, M), dtype=np.uint8), codes)
    return cw, np.ascontiguousarray(codes), np.ascontiguousarray(centers)


@pytest.mark.parametrize("M,N,K,kind", [
    (8, 30_001, 600, "wide"), (16, 30_001, 600, "wide"), (32, 30_001, 400, "wide"),      # more dimensions: left before the first scan
    (8, 30_001, 600, "ties"), (32, 30_001, 600, "ties"),                                 # too many centers alike in every block
    (8, 300_001, 1000, "some ties")])                                                    # 5 per code: only all blocks together are too much
def test_fit_that_is_left(env, M, N, K, kind):
    """The scans behind build their images over the points, and the iterations that follow start from them."""
    pq, oracle, torch = env
    rng = np.random.default_rng(M + N)
    if kind == "wide":
        cw, codes, centers = _problem(rng, N, M, K, 320 // M)
    else:
        cw, codes, centers = _alike(rng, N, M, K, 5 if kind == "some ties" else 200)
    t = oracle.build_tables(cw)
    iters = 1 if kind == "some ties" else 4
    c = torch.from_numpy(centers).cuda()
    h = torch.empty((K, M, 256), dtype=torch.int32, device="cuda")
    ws = torch.full((pq.workspace_bytes(N, M, K),), 0xA5, dtype=torch.uint8, device="cuda")
    pq.set_option("scan_variant", FORCED)
    try:
        _, a = pq.fit(torch.from_numpy(codes).cuda(), torch.from_numpy(t).cuda(), c, iters, hist=h, workspace=ws)
        assert pq.dot_scan(N, M, K, ws) == dict(tried=True, left=True)
    finally:
        pq.set_option("scan_variant", 0)
    want = centers
    for _ in range(iters):
        ra, _ = oracle.assign(codes, want, t)
        want, rh, _ = oracle.update(codes, ra, t, want)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(c.cpu().numpy(), want)
    np.testing.assert_array_equal(u32(h), rh)


def test_captured(env):
    """In a graph: kernels only, replayed with other work between."""
    pq, oracle, torch = env
    rng = np.random.default_rng(9)
    M, N, K = 16, 30_011, 300                      # a size at which the scan is chosen by itself
    cw, codes, centers = _problem(rng, N, M, K, 8)
    t = oracle.build_tables(cw)
    x, c, tt = (torch.from_numpy(v).cuda() for v in (codes, centers, t))
    ws = torch.empty(pq.workspace_bytes(N, M, K), dtype=torch.uint8, device="cuda")
    a = torch.empty(N, dtype=torch.int32, device="cuda")
    d = torch.empty(N, dtype=torch.float32, device="cuda")
    ra, rd = oracle.assign(codes, centers, t)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        pq.assign(x, c, tt, assign=a, dist=d, workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        pq.assign(x, c, tt, assign=a, dist=d, workspace=ws)
    for _ in range(3):
        a.fill_(-1)
        d.fill_(-1.0)
        ws.random_(0, 256)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(a.cpu().numpy(), ra)
        np.testing.assert_array_equal(d.cpu().numpy(), rd)
        assert pq.dot_scan(N, M, K, ws) == dict(tried=True, left=False)
