"""The scans through lower bounds against the oracle, where the bound, the candidates or the fall-back to the plain scan
can go wrong: edges of tiles and workgroups, ties, tables the bound says nothing about, non-finite and signed-zero entries,
several iterations from the centers of the one before."""
from __future__ import annotations

import numpy as np
import pytest

from _util import progress, rand_tables, u32

pytestmark = pytest.mark.gpu

VARIANTS = {4: [60, 61, 62, 63, 64], 8: [60, 61, 62, 63], 16: [59], 32: [59]}
ALL = [(M, v) for M in VARIANTS for v in VARIANTS[M]]


@pytest.fixture(scope="module")
def env():
    import torch

    import oracle
    import paper_1709_03708_amd as pq

    assert torch.cuda.is_available()
    return pq, oracle, torch


class _Variant:
    def __init__(self, pq, variant):
        self.pq, self.variant = pq, variant

    def __enter__(self):
        self.pq.set_option("assign_kernel", 2)
        self.pq.set_option("scan_variant", self.variant)

    def __exit__(self, *exc):
        self.pq.set_option("assign_kernel", 0)
        self.pq.set_option("scan_variant", 0)


def _check(env, codes, centers, tables, variant, offset=0):
    """offset: floats by which the tables are moved off their 16-byte alignment"""
    pq, oracle, torch = env
    N, M = codes.shape
    buf = torch.empty(tables.size + offset, dtype=torch.float32, device="cuda")
    t = buf[offset:].view(tables.shape)
    t.copy_(torch.from_numpy(tables))
    a = torch.full((N,), -7, dtype=torch.int32, device="cuda")
    d = torch.full((N,), float("nan"), dtype=torch.float32, device="cuda")
    with _Variant(pq, variant):
        # M = 16, 32: the byte tables need room for 65 centers
        assert pq.scan_plan(N, M, centers.shape[0])["scan"] == (2 if centers.shape[0] > {4: 0, 8: 16, 16: 64, 32: 64}[M] else 1)
        pq.assign(torch.from_numpy(codes).cuda(), torch.from_numpy(centers).cuda(), t, assign=a, dist=d)
    ra, rd = oracle.assign(codes, centers, tables)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    if M >= 16:      # may have been left to the sliding-window scan, whose minimum of a +0 and a -0 is either
        np.testing.assert_array_equal(d.cpu().numpy(), rd)
    else:
        np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), rd.view(np.uint32))


def _metric_tables(rng, M, dims=6):
    """dims: per subspace; M = 16 and 32: more than 256 in all are left by the scan on the matrix cores"""
    cw = rng.standard_normal((M, 256, dims)).astype(np.float32)
    return np.ascontiguousarray(((cw[:, :, None] - cw[:, None]) ** 2).sum(3, dtype=np.float32))


@pytest.mark.parametrize("M,variant", ALL)
@pytest.mark.parametrize("N,K", [(1, 1), (7, 64), (33, 63), (2047, 65), (2048, 128), (4097, 129), (2049, 66), (1025, 127), (4097, 191), (1024, 192),
                                 (20011, 640), (8191, 2000)])
def test_edges(env, M, variant, N, K):
    rng = np.random.default_rng(N + K + M)
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    near = centers[rng.integers(0, K, N)]
    codes = np.where(rng.random((N, M)) < 0.3, rng.integers(0, 256, (N, M)), near).astype(np.uint8)
    _check(env, codes, centers, _metric_tables(rng, M), variant, offset=N % 2)
    _check(env, codes, centers, rand_tables(rng, M), variant)                    # non-symmetric, no zero diagonal


def _special_tables(rng, M, kind):
    t = _metric_tables(rng, M)
    if kind == "constant":
        t[:] = 2.5
    elif kind == "zero":
        t[:] = 0.0
    elif kind == "signed zeros":
        t[:] = np.where(rng.random(t.shape) < 0.5, np.float32(0.0), np.float32(-0.0))
    elif kind == "hamming":
        t[:] = 1.0
        t[:, np.arange(256), np.arange(256)] = 0.0
    elif kind == "negative":
        t -= 40.0
    elif kind == "offset":
        t += np.float32(3e5)                       # spread far below the entries: sums tie by rounding
    elif kind == "outlier":
        t[0, 3, 5] = 1e30
        t[1, 7, 7] = -1e25
    elif kind == "huge":
        t *= np.float32(1e37)
    elif kind == "tiny":
        t *= np.float32(1e-42)
    elif kind == "non-finite":
        t[rng.random(t.shape) < 0.02] = np.nan
        t[rng.random(t.shape) < 0.02] = np.inf
    elif kind == "minus inf":
        t[rng.random(t.shape) < 0.001] = -np.inf
    elif kind == "nothing selected":
        t[0] = np.nan
        t[1] = np.inf
    return t


KINDS = ["constant", "zero", "signed zeros", "hamming", "negative", "offset", "outlier", "huge", "tiny", "non-finite", "minus inf",
         "nothing selected"]


@pytest.mark.parametrize("M,variant", [(M, v) for M, v in ALL if v in (61, 59, 64 if M == 4 else 63)])
@pytest.mark.parametrize("kind", KINDS)
def test_special_tables(env, M, variant, kind):
    rng = np.random.default_rng(len(kind) + M)
    N, K = 3001, 700
    centers = rng.integers(0, 40, (K, M), dtype=np.uint8)            # many equal centers
    codes = rng.integers(0, 40, (N, M), dtype=np.uint8)
    with np.errstate(all="ignore"):
        _check(env, codes, centers, _special_tables(rng, M, kind), variant)


@pytest.mark.parametrize("M,variant", [(M, v) for M, v in ALL if v in (60, 59, 64 if M == 4 else 63)])
@pytest.mark.parametrize("N,K,kind", [(30_011, 300, "metric"), (5003, 90, "hamming"), (5003, 90, "non-finite"), (9001, 400, "offset"),
                                      (3001, 200, "constant")])
def test_iterations(env, M, variant, N, K, kind):
    """Each iteration starts from the center of the one before; empty clusters, unchanged and changed centers among them."""
    pq, oracle, torch = env
    rng = np.random.default_rng(N + K)
    T = rng.integers(0, 256, (2 * K, M), dtype=np.uint8)
    codes = np.where(rng.random((N, M)) < 0.25, rng.integers(0, 256, (N, M)), T[rng.integers(0, 2 * K, N)]).astype(np.uint8)
    centers = codes[rng.integers(0, N, K)].copy()
    centers[K // 2] = centers[0]                                      # a center that stays empty
    with np.errstate(all="ignore"):
        tables = _metric_tables(rng, M) if kind == "metric" else _special_tables(rng, M, kind)
    d = dict(codes=torch.from_numpy(codes).cuda(), tables=torch.from_numpy(tables).cuda())
    for iters in (1, 2, 5):
        progress(f"lower-bound scan, {iters} iterations: M={M} variant={variant} N={N} K={K} {kind}")
        hist = torch.empty((K, M, 256), dtype=torch.int32, device="cuda")
        counts = torch.empty((K,), dtype=torch.int32, device="cuda")
        cent = torch.from_numpy(centers).cuda()
        with _Variant(pq, variant), np.errstate(all="ignore"):
            _, a = pq.fit(d["codes"], d["tables"], cent, iters, hist=hist, counts=counts)
        rc, ra, rh, rcnt = oracle.fit(codes, tables, centers, iters)
        np.testing.assert_array_equal(a.cpu().numpy(), ra)
        np.testing.assert_array_equal(u32(hist), rh)
        np.testing.assert_array_equal(u32(counts), rcnt)
        np.testing.assert_array_equal(cent.cpu().numpy(), rc)


@pytest.mark.parametrize("M,variant", [(M, v) for M, v in ALL if v in (59, 64 if M == 4 else 63)])
def test_launch_stretches(env, M, variant):
    """Several scan launches and rounds: keys by position serve one launch at a time, the bound then comes from assign[]."""
    pq, oracle, torch = env
    rng = np.random.default_rng(9)
    N, K = 70_003, 200
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    codes = np.where(rng.random((N, M)) < 0.3, rng.integers(0, 256, (N, M)), centers[rng.integers(0, K, N)]).astype(np.uint8)
    tables = _metric_tables(rng, M)
    rc, ra, _, _ = oracle.fit(codes, tables, centers, 3)
    try:
        pq.set_option("launch_codes_log2", 14)
        for forced in (0, 3):
            pq.set_option("hist_kernel", forced)
            cent = torch.from_numpy(centers).cuda()
            with _Variant(pq, variant):
                _, a = pq.fit(torch.from_numpy(codes).cuda(), torch.from_numpy(tables).cuda(), cent, 3)
            np.testing.assert_array_equal(a.cpu().numpy(), ra)
            np.testing.assert_array_equal(cent.cpu().numpy(), rc)
    finally:
        pq.set_option("launch_codes_log2", 26)
        pq.set_option("hist_kernel", 0)


@pytest.mark.parametrize("M,N,K,iters,launch,hist,dims", [
    (4, 1_834_980, 1000, 3, 21, 3, 6),       # first iteration in two stretches, second in one
    (4, 1_500_000, 600, 5, 26, 0, 6), (4, 700_000, 1000, 3, 26, 0, 6),
    (8, 4_200_000, 505, 5, 26, 0, 6),        # placed for four lanes first, read by two later
    (8, 4_200_000, 600, 5, 26, 0, 6), (8, 4_200_000, 950, 3, 26, 0, 6),
    (16, 400_000, 1000, 5, 26, 0, 18), (16, 400_000, 2000, 3, 26, 0, 18), (32, 270_000, 1600, 5, 26, 0, 10), (32, 270_000, 4100, 2, 26, 0, 10),
    (16, 400_000, 1000, 5, 26, 0, 6), (32, 270_000, 1600, 5, 26, 0, 6)])       # the scan on the matrix cores, in front of all of them
def test_plain_iterations_then_lower_bounds(env, M, N, K, iters, launch, hist, dims):
    """Default fits whose first iterations run a plain scan and whose later ones the lower-bound scan: what an iteration
    takes over from the one before (regrouped codes, statistics, keys) has to be there."""
    pq, oracle, torch = env
    rng = np.random.default_rng(M + K)
    centers = rng.integers(0, 256, (K, M), dtype=np.uint8)
    codes = centers[rng.integers(0, K, N)]
    fresh = rng.random((N, M), dtype=np.float32) < 0.3
    codes[fresh] = rng.integers(0, 256, int(fresh.sum()), dtype=np.uint8)
    tables = _metric_tables(rng, M, dims)
    progress(f"plain, then lower bounds: M={M} N={N} K={K} {dims} dimensions per subspace")
    try:
        pq.set_option("launch_codes_log2", launch)
        pq.set_option("hist_kernel", hist)
        assert pq.scan_plan(N, M, K, 0)["scan"] == 1 and pq.scan_plan(N, M, K, iters - 1)["scan"] == 2
        cent = torch.from_numpy(centers).cuda()
        a = torch.full((N,), -7, dtype=torch.int32, device="cuda")
        ws = torch.full((pq.workspace_bytes(N, M, K),), 0xA5, dtype=torch.uint8, device="cuda")
        pq.fit(torch.from_numpy(codes).cuda(), torch.from_numpy(tables).cuda(), cent, iters, assign=a, workspace=ws)
        torch.cuda.synchronize()
        assert pq.dot_scan(N, M, K, ws) == (dict(tried=True, left=dims * M > 256) if M >= 16 else dict(tried=False, left=None))
    finally:
        pq.set_option("launch_codes_log2", 26)
        pq.set_option("hist_kernel", 0)
    rc, ra, _, _ = oracle.fit(codes, tables, centers, iters)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(cent.cpu().numpy(), rc)


@pytest.mark.parametrize("M,variant", [(M, v) for M, v in ALL if v in (60, 59, 64 if M == 4 else 63)])
@pytest.mark.parametrize("hist_kernel", [0, 3])
def test_some_workgroups_give_up(env, M, variant, hist_kernel):
    """Stretches of codes that share no subcode with any center, between others that are close to one: the former tie with
    every center and are left to the plain scan, the latter are not, and both hand over to the histograms."""
    pq, oracle, torch = env
    rng = np.random.default_rng(M + hist_kernel)
    N, K = 60_013, 1100
    centers = rng.integers(0, 128, (K, M), dtype=np.uint8)
    codes = np.where(rng.random((N, M)) < 0.3, rng.integers(0, 128, (N, M)), centers[rng.integers(0, K, N)]).astype(np.uint8)
    codes[20_000:45_000] = 128 + (codes[20_000:45_000] & 3)
    tables = _metric_tables(rng, M)
    tables[:, 128:] = 50.0
    tables[:, :, 128:] = 50.0
    d = dict(codes=torch.from_numpy(codes).cuda(), tables=torch.from_numpy(tables).cuda())
    try:
        pq.set_option("hist_kernel", hist_kernel)
        for iters in (1, 4):
            hist = torch.empty((K, M, 256), dtype=torch.int32, device="cuda")
            cent = torch.from_numpy(centers).cuda()
            with _Variant(pq, variant):
                _, a = pq.fit(d["codes"], d["tables"], cent, iters, hist=hist)
            rc, ra, rh, _ = oracle.fit(codes, tables, centers, iters)
            np.testing.assert_array_equal(a.cpu().numpy(), ra)
            np.testing.assert_array_equal(u32(hist), rh)
            np.testing.assert_array_equal(cent.cpu().numpy(), rc)
    finally:
        pq.set_option("hist_kernel", 0)


@pytest.mark.parametrize("variant", [60, 63, 64])
def test_large_update_sorts_into_the_room_of_the_keys(env, variant):
    """M = 4 without records: the update of this size sorts the indices there, so the next iteration may not start from keys."""
    pq, _, torch = env
    g = torch.Generator(device="cuda")
    g.manual_seed(variant)
    N, M, K = 3_000_000, 4, 5000
    T = torch.randint(0, 256, (K, M), generator=g, device="cuda", dtype=torch.uint8)
    x = T[torch.randint(0, K, (N,), generator=g, device="cuda")]
    x = torch.where(torch.rand(N, M, generator=g, device="cuda") < 0.3,
                    torch.randint(0, 256, (N, M), generator=g, device="cuda", dtype=torch.uint8), x).contiguous()
    t = pq.build_tables(torch.randn(M, 256, 8, generator=g, device="cuda"))
    out = []
    for v in (variant, 65):                                           # 65: plain scans
        c = x[:K].clone()
        with _Variant(pq, v):
            if v == variant:
                assert pq.scan_plan(N, M, K, 2)["seeded"] == (2 if v == 63 else 1)
            _, a = pq.fit(x, t, c, 3)
        out.append((a, c))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("M,N,K,late", [(32, 270_000, 1700, False), (32, 270_000, 1700, True), (16, 395_000, 2300, True), (16, 395_000, 2300, False)])
def test_wide_scan_in_several_launches(env, M, N, K, late):
    """More than one round of workgroups, so that the tiles come in several launches: keys and counts of candidates carry over.
    late: the centers of the last tiles are all at the same distance from many codes, so that workgroups give up in a launch
    after others have carried their keys over or have written results."""
    pq, oracle, torch = env
    rng = np.random.default_rng(M + late)
    centers = rng.integers(0, 128, (K, M), dtype=np.uint8)
    codes = centers[rng.integers(0, K // 2, N)]
    fresh = rng.random((N, M), dtype=np.float32) < 0.5
    codes[fresh] = rng.integers(0, 128, int(fresh.sum()), dtype=np.uint8)
    tables = _metric_tables(rng, M)
    if late:
        tables[:, :, 200] = tables[:, :, :128].min(axis=2) * np.float32(0.5)      # near every code in every subspace
        centers[K // 2 + 64:] = 200
    a = torch.full((N,), -7, dtype=torch.int32, device="cuda")
    d = torch.full((N,), float("nan"), dtype=torch.float32, device="cuda")
    progress(f"wide scan, several launches: M={M} N={N} K={K} late={late}")
    with _Variant(pq, 59):
        pq.assign(torch.from_numpy(codes).cuda(), torch.from_numpy(centers).cuda(), torch.from_numpy(tables).cuda(), assign=a, dist=d)
    ra, rd = oracle.assign(codes, centers, tables)
    np.testing.assert_array_equal(a.cpu().numpy(), ra)
    np.testing.assert_array_equal(d.cpu().numpy(), rd)


@pytest.mark.parametrize("M,N,K,plain", [(4, 1_000_000, 4000, 65), (4, 3_000_000, 10_000, 65), (8, 4_300_000, 2000, 80), (16, 500_000, 4000, 50),
                                         (32, 300_000, 10_000, 50)])
@pytest.mark.parametrize("kind", ["constant", "hamming"])
def test_giving_up_costs_little(env, M, N, K, plain, kind):
    """Tables that the bounds say nothing or too little about: the time stays near that of the plain scan (it was up to ten
    times that)."""
    pq, _, torch = env
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    codes = torch.randint(0, 256, (N, M), generator=g, device="cuda", dtype=torch.uint8)
    centers = torch.randint(0, 256, (K, M), generator=g, device="cuda", dtype=torch.uint8)
    tables = torch.ones(M, 256, 256, device="cuda")
    if kind == "hamming":
        tables[:, torch.arange(256), torch.arange(256)] = 0.0
    ws = torch.empty(pq.workspace_bytes(N, M, K), dtype=torch.uint8, device="cuda")
    out = {}
    for variant in (0, plain):
        a = torch.empty(N, dtype=torch.int32, device="cuda")
        times = []
        pq.set_option("scan_variant", variant)
        try:
            for _ in range(4):
                s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                s.record()
                pq.assign(codes, centers, tables, assign=a, want_dist=False, workspace=ws)
                e.record()
                torch.cuda.synchronize()
                times.append(s.elapsed_time(e))
        finally:
            pq.set_option("scan_variant", 0)
        out[variant] = (min(times), a)
    assert torch.equal(out[0][1], out[plain][1])
    assert out[0][0] < 2.2 * out[plain][0]                   # measured 1.0 to 1.7


@pytest.mark.parametrize("M,N,K,dims", [(4, 600_000, 2000, 8), (32, 300_000, 5200, 8), (32, 300_000, 5200, 12), (16, 400_000, 4000, 20)])
def test_captured_fit(env, M, N, K, dims):
    """dims: per subspace; more than 256 in all are left by the scan on the matrix cores.  The default scans of these sizes in a captured graph, with eager work and another workspace content between replays."""
    pq, _, torch = env
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    T = torch.randint(0, 256, (2 * K, M), generator=g, device="cuda", dtype=torch.uint8)
    codes = T[torch.randint(0, 2 * K, (N,), generator=g, device="cuda")]
    fresh = torch.randint(0, 256, (N, M), generator=g, device="cuda", dtype=torch.uint8)
    codes = torch.where(torch.rand(N, M, generator=g, device="cuda") < 0.2, fresh, codes).contiguous()
    cent0 = codes[:K].clone()
    tables = pq.build_tables(torch.randn(M, 256, dims, generator=g, device="cuda"))
    ws = torch.empty(pq.workspace_bytes(N, M, K), dtype=torch.uint8, device="cuda")
    eager, a0 = cent0.clone(), torch.full((N,), -1, dtype=torch.int32, device="cuda")
    pq.fit(codes, tables, eager, 4, assign=a0, workspace=ws)
    torch.cuda.synchronize()
    cent, a = cent0.clone(), torch.full((N,), -1, dtype=torch.int32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pq.fit(codes, tables, cent, 4, assign=a, workspace=ws)
    for rep in range(3):
        cent.copy_(cent0)
        a.fill_(-1)
        ws.fill_(rep + 3)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(cent, eager) and torch.equal(a, a0), f"replay {rep}"
        assert pq.dot_scan(N, M, K, ws) == (dict(tried=True, left=dims * M > 256) if M >= 16 else dict(tried=False, left=None))
