"""Which scan the iterations of a fit run, and what one takes over from the one before (host arithmetic, no GPU): the
regrouped copy of the codes may only be taken over when the iteration that made it covered all codes in one stretch and
placed them for the slots that read it; keys by position only together with that copy."""
from __future__ import annotations

import random

import pytest


@pytest.fixture(scope="module")
def pq():
    import os

    import paper_1709_03708_amd as pq

    if not os.path.exists(pq.lib_path()):
        from paper_1709_03708_amd import build

        build.build()
    return pq


def _walk(pq, N, M, K, iters):
    copy, lanes, before = 0, 0, None              # codes covered by the copy in one stretch, its layout, the plan before
    seen = []
    for it in range(iters):
        p = pq.scan_plan(N, M, K, it)
        if p["lanes"]:
            if p["reuse"]:
                assert copy == N and lanes == p["lanes"] and p["per_launch"] >= N, (N, M, K, it, p, before)
            else:
                copy, lanes = (N if N <= p["per_launch"] else 0), p["lanes"]
        else:
            assert not p["reuse"]
            copy = 0
        if p["scan"] == 2 and M <= 8:
            assert (it == 0) == (p["seeded"] in (0, 3)), (N, M, K, it, p)
            if p["seeded"] == 2:
                assert p["reuse"] and before["scan"] == 2 and before["variant"] == p["variant"], (N, M, K, it, p, before)
        before = p
        seen.append(p)
    return seen


def _options(pq, launch=26, hist=0, variant=0):
    pq.set_option("launch_codes_log2", launch)
    pq.set_option("hist_kernel", hist)
    pq.set_option("scan_variant", variant)


@pytest.fixture(autouse=True)
def defaults(pq):
    yield
    _options(pq)


def test_stretch_lengths_that_differ_between_iterations(pq):
    """A plain scan in two stretches, then the lower-bound scan in one: the copy of the first is not all of the codes."""
    _options(pq, launch=21, hist=3)
    N, K = 1_834_980, 1000
    first, second, third = _walk(pq, N, 4, K, 3)
    assert first["scan"] == 1 and first["per_launch"] < N
    assert second["scan"] == 2 and second["per_launch"] >= N and not second["reuse"]
    assert third["reuse"]


@pytest.mark.parametrize("launch", [20, 21, 22, 23, 24, 26])
@pytest.mark.parametrize("hist", [0, 1, 2, 3])
def test_takeover_near_every_stretch_length(pq, launch, hist):
    """N around the stretch length of every iteration's scan, where one iteration needs more stretches than another."""
    _options(pq, launch, hist)
    for M, Ks in ((4, (400, 500, 700, 900, 1000, 1799, 1800, 5000)), (8, (256, 500, 505, 511, 512, 700, 900, 1799, 1800))):
        for K in Ks:
            N = 1 << launch
            lengths = {pq.scan_plan(n, M, K, it)["per_launch"] for n in (N // 2, 3 * N // 4, N) for it in (0, 1, 3)}
            for length in lengths:
                for d in (-33, -17, -1, 0, 1, 4, 16, 33):
                    if length + d > 0:
                        _walk(pq, length + d, M, K, 5)


def test_takeover_over_random_sizes(pq):
    rng = random.Random(1)
    for _ in range(3000):
        _options(pq, rng.choice([12, 16, 20, 21, 22, 23, 24, 26, 30]), rng.randrange(4), rng.choice([0, 0, 0, 60, 62, 65, 70, 80, 85]))
        N = int(2 ** rng.uniform(0, 27)) + rng.randrange(40)
        _walk(pq, N, rng.choice([4, 8, 16, 32]), int(2 ** rng.uniform(0, 16)), 5)


@pytest.mark.parametrize("M,N,K", [(8, 4_300_000, 505), (8, 4_300_000, 1000), (4, 3_000_000, 1000)])
def test_copy_is_placed_for_the_scan_that_reads_it(pq, M, N, K):
    """Plain scans of the first iterations may place the codes for four lanes; the lower-bound scan reads them with two."""
    plans = _walk(pq, N, M, K, 6)
    assert plans[0]["scan"] == 1 and plans[-1]["scan"] == 2
    assert plans[-1]["lanes"] == 2 and plans[-1]["reuse"] and plans[-1]["seeded"] == 2


@pytest.mark.parametrize("M,K,most", [(4, 16, 4700), (4, 64, 9400), (4, 100, 16384), (8, 16, 7800), (8, 100, 16384), (16, 3, 11600), (32, 1, 16384)])
def test_few_codes_take_no_more_than_a_round_of_tiles(pq, M, K, most):
    """One lane per center only up to the codes for which it is the faster one: with few centers the tiled scans are cheap."""
    assert pq.scan_plan(most, M, K)["scan"] == 0 and pq.scan_plan(most + 1, M, K)["scan"] == 1


def test_matrix_core_scan_where_it_is_built(pq):
    """M = 4 has no scan on the matrix cores, and one that regroups its codes is not preceded by it."""
    _options(pq, variant=20)
    assert not pq.dot_scan(100_000, 4, 1000)["tried"]
    assert not pq.dot_scan(100_000, 8, 16)["tried"] and pq.dot_scan(100_000, 8, 17)["tried"]      # the images leave no room for it
    assert pq.dot_scan(100_000, 16, 1)["tried"] and pq.dot_scan(100_000, 32, 1)["tried"]
    assert not pq.dot_scan(5_000_000, 8, 1000)["tried"] and pq.scan_plan(5_000_000, 8, 1000)["lanes"]
    _options(pq)


@pytest.mark.parametrize("M,N,K", [(8, 180_000, 500), (16, 140_626, 64), (16, 764_706, 17), (32, 562_501, 16), (16, 25_000, 360)])
def test_matrix_core_scan_by_size(pq, M, N, K):
    """Edges of the rule: one code or center less and the plain scans run alone."""
    assert pq.dot_scan(N, M, K)["tried"] and pq.scan_plan(N, M, K)["scan"] == 1
    assert not pq.dot_scan(N, M, K - 1)["tried"]
    assert not pq.dot_scan(N - 2, M, K)["tried"]


def test_one_lane_per_center_comes_before_the_matrix_core_scan(pq):
    for M, N, K in ((32, 47_058, 1000), (16, 86_486, 4000), (8, 86_486, 4000)):
        assert not pq.dot_scan(N, M, K)["tried"] and pq.scan_plan(N, M, K)["scan"] == 0
        assert pq.dot_scan(N + 1, M, K)["tried"]


@pytest.mark.parametrize("variant,seeded", [(0, 2), (60, 1), (61, 1), (62, 1), (63, 2), (64, 1)])
def test_keys_share_their_room_with_the_sorted_indices(pq, variant, seeded):
    """Of the M = 4 scans through lower bounds only 63 files records; behind the others a large update sorts the indices into the
    room of the keys, and the next iteration starts from assign[]."""
    _options(pq, variant=variant)
    assert pq.scan_plan(3_000_000, 4, 5000, 2)["seeded"] == seeded
    _options(pq, variant=variant, hist=2)
    assert pq.scan_plan(3_000_000, 4, 5000, 2)["seeded"] == 2
