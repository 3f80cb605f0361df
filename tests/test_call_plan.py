"""What one assignment and one update by themselves run, by size, alignment and options (host arithmetic, no GPU: the answers are
those for 256 compute units)."""
from __future__ import annotations

import os

import pytest


@pytest.fixture(scope="module")
def pq():
    import torch

    import paper_1709_03708_amd as pq

    if not os.path.exists(pq.lib_path()):
        from paper_1709_03708_amd import build

        build.build()
    if torch.cuda.is_available() and torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rules count compute units")
    return pq


def test_arguments(pq):
    import ctypes

    out = (ctypes.c_int64 * 8)()
    call = pq.load().pqkm_call_plan
    assert call(10, 4, 10, 0, None) == 1
    for bad in ((-1, 4, 10, 0), (10, 65, 10, 0), (10, 4, 0, 0), (10, 4, 10, 8), (10, 4, 10, -1)):
        assert call(*bad, out) == 2
    assert call(0, 4, 10, 7, out) == 0


@pytest.mark.parametrize("N,K,variant", [(655_360, 64, 38), (786_000, 40, 39), (1_000_000, 32, 37), (786_433, 100, 34), (600_001, 300, 38)])
def test_skewed_shapes(pq, N, K, variant):
    """M = 4, few centers: the shape whose rounds take least; beyond 127 centers only for one assignment by itself."""
    p = pq.call_plan(N, 4, K)
    assert p["scan"] == "tiled" and p["variant"] == variant
    if K < 128:
        assert pq.scan_plan(N, 4, K)["variant"] == variant
    else:
        assert pq.scan_plan(N, 4, K)["variant"] != variant


@pytest.mark.parametrize("M,N,K,dims", [(8, 36_001, 1000, 128), (8, 20_000, 1000, 0), (16, 24_000, 300, 128), (16, 9000, 300, 0),
                                        (16, 30_011, 1000, 256), (32, 11_003, 1500, 128), (32, 5000, 160, 0), (4, 46_000, 1000, 0)])
def test_matrix_cores_before_one_lane_per_center(pq, M, N, K, dims):
    """pqkm_dot_scan answers for the scans behind the tiled sizes only."""
    p = pq.call_plan(N, M, K)
    assert p["scan"] == "one_lane_per_center" and p["dot"] == dims
    assert not pq.dot_scan(N, M, K)["tried"]


def test_matrix_cores_with_more_centers_than_codes(pq):
    """They lie close together: not for a small gain."""
    assert pq.call_plan(8000, 16, 50_000)["dot"] == 0 and pq.call_plan(8000, 32, 20_000)["dot"] > 0


@pytest.mark.parametrize("M,K,least", [(4, 300, 19_459), (4, 1000, 47_058), (8, 1000, 47_058), (8, 4000, 86_486), (16, 300, 19_459), (32, 300, 19_459)])
def test_centers_off_their_alignment(pq, M, K, least):
    """They are read byte by byte, which is slower than the tiled scans from fewer codes on."""
    assert pq.call_plan(least, M, K, centers_aligned=False)["scan"] == "one_lane_per_center"
    p = pq.call_plan(least + 1, M, K, centers_aligned=False)
    assert p["scan"] == "tiled" and p["dot"] == 0
    if M == 4:
        assert pq.call_plan(least + 1, M, K)["scan"] == "one_lane_per_center"


@pytest.mark.parametrize("M,N,K,codes", [(4, 1, 2500, 1), (4, 257, 300_000, 0), (4, 1025, 300_000, 0), (4, 2100, 50_000, 0), (8, 257, 300_000, 0), (8, 2100, 50_000, 0),
                                         (16, 257, 50_000, 0), (16, 8000, 1000, 2), (16, 8000, 300, 1), (32, 257, 50_000, 1), (32, 1025, 50_000, 1),
                                         (4, 8000, 1000, 4)])
def test_blocks_of_one_lane_per_center(pq, M, N, K, codes):
    """Blocks fill the compute units evenly: a code more than one block per unit takes may not double the time."""
    p = pq.call_plan(N, M, K)
    assert p["scan"] == "one_lane_per_center" and p["variant"] == 1
    assert p["codes"] == codes or not codes
    passes, blocks = -(-K // 256), -(-N // p["codes"]) * p["parts"]
    if passes * M > 700:
        assert -(-passes // p["parts"]) * -(-blocks // 256) * p["codes"] < 1.35 * passes * N / 256          # the busiest unit's passes over a code
    else:
        assert p["parts"] == 1
    for n, k in ((N, K), (N + 1, K), (2 * N, K), (N, 2 * K)):
        q = pq.call_plan(n, M, k)
        if q["scan"] == "one_lane_per_center":
            assert q["parts"] == 1 or q["parts"] * n * 8 <= (k + 128 // M - 1) // (128 // M) * 131072      # their records fit the images' room
    assert pq.call_plan(N, M, 95)["variant"] == (1 if M < 16 else 0)


def test_rows_of_sixteen_subspaces(pq):
    assert pq.call_plan(2000, 16, 95)["variant"] == 0 and pq.call_plan(2000, 16, 96)["variant"] == 1


@pytest.mark.parametrize("M,N,K,aligned,few", [(4, 40_000, 16, True, True), (4, 40_001, 16, True, False), (4, 28_000, 8, True, True), (4, 28_001, 8, True, False), (8, 20_000, 3, True, True), (8, 20_001, 3, True, False),
                                               (4, 40_000, 256, True, True), (4, 40_000, 257, True, False), (64, 40_000, 8, True, False),
                                               (6, 12_000, 85, True, True), (6, 12_000, 86, True, False), (6, 1499, 128, True, True), (4, 12_001, 16, False, False)])
def test_vote_that_counts_a_cluster_per_workgroup(pq, M, N, K, aligned, few):
    """Not where a workgroup has too large a share of the codes, or reads four subspaces of them byte by byte."""
    assert (pq.call_plan(N, M, K, codes_aligned=aligned)["count"] == "vote_per_cluster") == few


@pytest.mark.parametrize("M,N,K,few", [(4, 47_500, 1000, True), (4, 100_000, 1000, False), (8, 50_000, 500, False), (8, 50_000, 300, True), (6, 300_000, 300, False),
                                       (6, 300_000, 200, True), (6, 60_000, 3000, True), (6, 10_000, 3001, False), (4, 100_000, 10_000, True), (8, 20_000, 5000, True),
                                       (8, 20_000, 5001, False), (16, 20_000, 2250, True), (16, 20_000, 2251, False), (32, 10_000, 5000, False), (64, 5000, 1000, True),
                                       (64, 5000, 1001, False), (2, 200_000, 1000, True), (3, 500_000, 700, True), (4, 500_000, 512, True), (4, 500_000, 513, False),
                                       (8, 500_000, 256, True), (8, 500_000, 257, False), (5, 400_000, 257, False)])
def test_vote_with_a_workgroup_per_cluster(pq, M, N, K, few):
    assert pq.call_plan(N, M, K)["vote_per_cluster"] == few


def test_partial_histograms_of_subspaces_have_a_vote_that_adds_them(pq):
    """Up to 64 arrays of 16-bit counters: only the vote with a workgroup per cluster reads them."""
    import random

    rng = random.Random(1)
    seen = 0
    for _ in range(20_000):
        M, K, N = rng.randint(1, 64), int(2 ** rng.uniform(0, 7.1)), int(2 ** rng.uniform(17, 25))
        p = pq.call_plan(N, M, K)
        if p["count"] == "subspaces":
            seen += 1
            assert p["vote_per_cluster"], (M, N, K)
        assert p["slices"] <= (64 if p["vote_per_cluster"] else 16)
    assert seen > 1000


@pytest.mark.parametrize("M,N,K,by_group", [(4, 100_000, 3000, True), (12, 1_000_000, 1333, True), (24, 400_000, 333, True), (40, 100_000, 400, True), (48, 100_000, 166, True),
                                            (4, 100_000, 2000, True), (4, 299_999, 2000, True), (4, 1_500_000, 2000, True), (8, 2_000_000, 5000, True), (16, 100_000, 500, True),
                                            (16, 800_000, 300, True), (32, 100_000, 150, True), (64, 100_000, 75, True),
                                            (4, 99_999, 3000, False), (4, 300_000, 2000, False), (8, 1_000_000, 1000, False), (16, 100_000, 300, False), (12, 200_000, 1000, False),
                                            (12, 100_000, 2000, False), (20, 400_000, 400, False), (24, 100_000, 200, False), (48, 100_000, 100, False),
                                            (48, 100_000, 500, False), (6, 300_000, 1000, False), (8, 201_135, 4060, False), (16, 224_433, 1737, False),
                                            (32, 299_108, 805, True), (56, 232_257, 133, False)])
def test_sort_by_group(pq, M, N, K, by_group):
    """Not where clusters of nearly even size lose by it: a last round of the owner path that is full, and groups that leave counters unused."""
    assert pq.call_plan(N, M, K)["count"] == ("sorted" if by_group else "cluster_groups")


@pytest.mark.parametrize("M,N,K,dims", [(8, 56_000, 300, 0), (8, 50_000, 400, 128), (8, 62_000, 400, 0), (8, 60_000, 512, 128), (16, 28_000, 160, 128), (16, 36_000, 160, 0),
                                        (16, 41_000, 200, 0), (16, 35_000, 256, 256), (32, 34_000, 160, 256), (32, 38_000, 160, 0), (32, 39_000, 230, 256)])
def test_matrix_cores_where_being_left_costs_no_more_than_tiles(pq, M, N, K, dims):
    """Tables they are not for pay 10 to 14 us to be told so, in front of one lane per center."""
    p = pq.call_plan(N, M, K)
    assert p["scan"] == "one_lane_per_center" and p["dot"] == dims


@pytest.mark.parametrize("M,K,most", [(4, 160, 41_111), (4, 200, 53_209), (4, 300, 63_911), (8, 160, 37_379), (8, 200, 46_151), (8, 300, 56_543)])
def test_limit_of_rows_with_one_pass(pq, M, K, most):
    """A block's only pass takes hardly less with fewer centers."""
    assert pq.call_plan(most, M, K)["scan"] == "one_lane_per_center" and pq.call_plan(most + 1, M, K)["scan"] == "tiled"


@pytest.mark.parametrize("M,N,K,taken", [(4, 1_000_000, 100, True), (4, 999_999, 100, False), (4, 1_200_000, 32, True), (4, 1_199_999, 32, False), (8, 1_000_000, 48, True),
                                         (12, 1_499_999, 32, False), (12, 1_500_000, 32, True), (8, 1_700_000, 100, True), (8, 1_600_000, 128, False), (8, 2_200_000, 128, True),
                                         (16, 1_600_000, 64, False), (16, 2_200_000, 64, True), (17, 4_000_000, 33, False), (32, 1_000_000, 20, True),
                                         (4, 2_000_000, 31, False)])
def test_histograms_by_subspace(pq, M, N, K, taken):
    """Enough slices to fill the chip, and codes to pay for adding their arrays."""
    assert (pq.call_plan(N, M, K)["count"] == "subspaces") == taken


@pytest.mark.parametrize("M,N,K,codes,parts", [(4, 48, 7936, 1, 1), (4, 48, 15_872, 2, 32), (4, 256, 15_872, 1, 1), (4, 256, 63_488, 2, 4), (4, 257, 63_488, 2, 16),
                                               (8, 1, 6913, 1, 1), (8, 1, 13_824, 1, 54), (8, 256, 13_824, 1, 1), (8, 257, 13_824, 1, 6), (16, 48, 3841, 1, 1),
                                               (16, 48, 7680, 1, 16), (16, 257, 7680, 1, 6), (32, 48, 1793, 1, 1), (32, 48, 3584, 1, 14), (32, 257, 14_336, 1, 8)])
def test_blocks_of_a_code_per_unit(pq, M, N, K, codes, parts):
    """Up to a block per compute unit there is nothing to choose until the centers take long enough to split."""
    p = pq.call_plan(N, M, K)
    assert (p["codes"], p["parts"]) == (codes, parts)


@pytest.mark.parametrize("M,N,K", [(48, 1_050_287, 1), (48, 2_501_840, 7), (40, 1_928_309, 2), (40, 2_036_211, 20), (20, 2_000_000, 20), (12, 2_000_000, 40), (5, 1_500_000, 40),
                                   (4, 1_000_000, 100)])
def test_slices_of_subspace_groups_share_a_die(pq, M, N, K):
    """Workgroups of different subspaces read the same codes: through one L2 only where the slices are a multiple of eight."""
    p = pq.call_plan(N, M, K)
    assert p["count"] == "subspaces" and p["slices"] > 8
    width = next(g for g in (4, 2, 1) if g == 1 or (g <= M and K * 256 * g <= 32768))
    assert p["slices"] % 8 == 0 or width >= M
