"""Encoder and decoder against the oracle where their kernels can go wrong: every padding of the subvector length, the
edges of the 32-vector tiles, ties, near ties, unaligned and non-finite inputs, extreme scales."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    import oracle
    import paper_1709_03708_amd as pq

    assert torch.cuda.is_available()
    return pq, oracle, torch


def _encode(env, vectors, cw, offset=0):
    pq, _, torch = env
    buf = torch.empty(vectors.size + offset, dtype=torch.float32, device="cuda")
    v = buf[offset:].view(vectors.shape)
    v.copy_(torch.from_numpy(vectors))
    return pq.encode(v, torch.from_numpy(cw).cuda()).cpu().numpy()


@pytest.mark.parametrize("M,Ds,N", [(1, 1, 1), (3, 3, 33), (16, 6, 65), (8, 12, 1000), (4, 16, 31), (5, 20, 97), (4, 24, 513),
                                    (4, 32, 2049), (9, 33, 64), (3, 48, 100), (2, 64, 3000), (2, 100, 95), (32, 128, 70),
                                    (2, 130, 40)])
@pytest.mark.parametrize("offset", [0, 1])
def test_encode_paddings_and_edges(env, M, Ds, N, offset):
    oracle = env[1]
    rng = np.random.default_rng(M * 1000 + Ds)
    cw = np.abs(20 * rng.standard_normal((M, 256, Ds))).astype(np.float32)
    vectors = np.abs(20 * rng.standard_normal((N, M * Ds))).astype(np.float32)
    assert np.array_equal(_encode(env, vectors, cw, offset), oracle.encode(vectors, cw))


@pytest.mark.parametrize("Ds", [4, 12, 32, 128])
def test_encode_ties_and_near_ties(env, Ds):
    """Duplicated codewords (the lower index wins), codewords one rounding apart, and vectors half-way between two."""
    oracle = env[1]
    rng = np.random.default_rng(Ds)
    M, N = 2, 700
    cw = rng.standard_normal((M, 256, Ds)).astype(np.float32)
    cw[:, 128:192] = cw[:, :64]
    cw[:, 192:224] = np.nextafter(cw[:, 64:96], np.float32(9))
    cw[:, 224:240] = cw[:, 5:6]
    vectors = rng.standard_normal((N, M, Ds)).astype(np.float32)
    for n in range(0, N, 2):
        a, b = rng.integers(0, 256, 2)
        vectors[n] = (cw[:, a] + cw[:, b]) * np.float32(0.5)
    for n in range(1, N, 4):
        vectors[n] = cw[:, rng.integers(0, 256)]
    vectors = vectors.reshape(N, M * Ds)
    assert np.array_equal(_encode(env, vectors, cw), oracle.encode(vectors, cw))


@pytest.mark.parametrize("scale", [1e-42, 1e-30, 1e-19, 1e-12, 1e12, 1e18, 3e37])
@pytest.mark.parametrize("shift", [0.0, 1000.0])
def test_encode_scales(env, scale, shift):
    """Squares that underflow, products that overflow, and a common offset far larger than the distances."""
    oracle = env[1]
    rng = np.random.default_rng(3)
    with np.errstate(over="ignore", under="ignore"):
        cw = ((rng.standard_normal((2, 256, 16)) + shift) * scale).astype(np.float32)
        vectors = ((rng.standard_normal((300, 32)) + shift) * scale).astype(np.float32)
    assert np.array_equal(_encode(env, vectors, cw), oracle.encode(vectors, cw))


def test_encode_non_finite(env):
    oracle = env[1]
    rng = np.random.default_rng(4)
    cw = rng.standard_normal((3, 256, 24)).astype(np.float32)
    vectors = rng.standard_normal((200, 72)).astype(np.float32)
    vectors[3, 5] = np.nan
    vectors[64, 30] = np.inf
    vectors[65, 30] = -np.inf
    vectors[199] = np.nan
    cw[1, 7, 3] = np.inf
    cw[2, 0] = np.nan
    cw[2, 9, 1] = 3e38
    assert np.array_equal(_encode(env, vectors, cw), oracle.encode(vectors, cw))


@pytest.mark.parametrize("M,Ds,N", [(1, 1, 1), (1, 1, 4099), (5, 3, 17), (16, 6, 1001), (8, 12, 999), (8, 16, 4096), (4, 32, 1),
                                    (32, 128, 33), (3, 130, 50), (7, 7, 2048)])
@pytest.mark.parametrize("offset", [0, 1])
def test_decode_shapes(env, M, Ds, N, offset):
    pq, oracle, torch = env
    rng = np.random.default_rng(M + Ds)
    cw = rng.standard_normal((M, 256, Ds)).astype(np.float32)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    buf = torch.full((N * M * Ds + offset + 64,), -7.0, device="cuda")
    out = buf[offset:offset + N * M * Ds].view(N, M * Ds)
    pq.decode(torch.from_numpy(codes).cuda(), torch.from_numpy(cw).cuda(), vectors=out)
    assert np.array_equal(out.cpu().numpy(), oracle.decode_f32(cw, codes))
    assert bool((buf[offset + N * M * Ds:] == -7.0).all()) and bool((buf[:offset] == -7.0).all())


@pytest.mark.parametrize("M,Ds", [(1, 4), (3, 16), (2, 40)])
def test_encode_distances_that_overflow(env, M, Ds):
    """Squares that are finite, distances that are not: where every distance is +inf the code is 0, where some are finite it
    is the closest of those."""
    oracle = env[1]
    rng = np.random.default_rng(Ds)
    with np.errstate(over="ignore"):
        cw = (-(0.5 + rng.random((M, 256, Ds))) * 1.5e19 / np.sqrt(Ds)).astype(np.float32)
        cw[-1, 17] = np.float32(1e18)                                     # one codeword within reach of the last subspace
        vectors = ((0.8 + 0.3 * rng.random((200, M, Ds))) * 1.5e19 / np.sqrt(Ds)).astype(np.float32)
        vectors[50:100] *= np.float32(0.01)
        vectors = vectors.reshape(200, M * Ds)
        assert np.array_equal(_encode(env, vectors, cw), oracle.encode(vectors, cw))


@pytest.mark.parametrize("Ds", [16, 96, 128])
def test_encode_codewords_on_a_sphere(env, Ds):
    """Vectors much shorter than codewords of nearly equal length: the matrix cores' sums start at the codeword's half
    square and stay as large, and the distances differ by less than their rounding."""
    oracle = env[1]
    rng = np.random.default_rng(Ds)
    cw = rng.standard_normal((2, 256, Ds))
    cw = (cw / np.linalg.norm(cw, axis=2, keepdims=True)).astype(np.float32)
    for size in (1e-6, 1e-5, 1e-4, 1e-3):
        vectors = (size * rng.standard_normal((500, 2 * Ds))).astype(np.float32)
        assert np.array_equal(_encode(env, vectors, cw), oracle.encode(vectors, cw))


@pytest.mark.parametrize("M,Ds,N", [(3, 1, 4000), (2, 4, 70_000), (5, 7, 6000), (2, 16, 40_000), (1, 33, 9000), (2, 64, 20_000), (1, 100, 3000)])
@pytest.mark.parametrize("kind", ["offset", "two clusters", "few of them open"])
def test_encode_open_vectors(env, M, Ds, N, kind):
    """Data whose gaps are small against their size or their spread, with the tiles of 32 in every state: all open, some, none;
    enough of them that a wave goes on after tiles it had to settle on the vector units."""
    oracle = env[1]
    rng = np.random.default_rng(Ds + N)
    cw = rng.standard_normal((M, 256, Ds))
    vectors = rng.standard_normal((N, M, Ds))
    if kind == "offset":
        cw, vectors = cw + 1000.0, vectors + 1000.0
    elif kind == "two clusters":
        cw += 300.0 * (rng.random((M, 256, 1)) < 0.5)
        vectors += 300.0 * (rng.random((N, M, 1)) < 0.5)
    else:
        cw[:, ::2] = cw[:, 1::2]                                       # every codeword twice
        cw[:, 64:128] *= 1e3
        vectors[rng.random(N) < 0.1] *= 1e3
    cw, vectors = cw.astype(np.float32), vectors.astype(np.float32).reshape(N, M * Ds)
    assert np.array_equal(_encode(env, vectors, cw), oracle.encode(vectors, cw))
    assert np.array_equal(_encode(env, vectors[: N // 3], cw, 1), oracle.encode(vectors[: N // 3], cw))


def test_encode_time_does_not_depend_on_a_common_offset(env):
    """The share of open vectors, and with it the time, is that of the centred data."""
    pq, _, torch = env
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    v = torch.randn(300_000, 128, generator=g, device="cuda")
    cw = torch.randn(4, 256, 32, generator=g, device="cuda")

    def best_us(shift):
        a, b = v + shift, cw + shift
        times = []
        for _ in range(5):
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s.record()
            pq.encode(a, b)
            e.record()
            torch.cuda.synchronize()
            times.append(s.elapsed_time(e) * 1e3)
        return min(times)

    assert best_us(100.0) < 3.0 * best_us(0.0)                         # 13 times before the data were centred


@pytest.mark.parametrize("M,Ds,N", [(3, 7, 199_728), (3, 7, 199_729), (5, 6, 139_811), (16, 3, 100_001), (32, 9, 14_600), (1, 1, 4_194_307),
                                    (2, 1001, 2200)])
def test_decode_odd_lengths(env, M, Ds, N):
    """Both sides of the sizes from which a thread writes four elements of an odd length, and ragged ends of those."""
    pq, oracle, torch = env
    rng = np.random.default_rng(N)
    cw = rng.standard_normal((M, 256, Ds)).astype(np.float32)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    got = pq.decode(torch.from_numpy(codes).cuda(), torch.from_numpy(cw).cuda()).cpu().numpy()
    assert np.array_equal(got, cw[np.arange(M), codes].reshape(N, M * Ds))
