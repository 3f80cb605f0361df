"""The encoder for subvectors of up to 8 dimensions, whose three products and norm share one or two matrix instructions: every
length and its neighbours in the padded ones, both alignments, ties, equal lengths, and values that overflow or are none."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(vectors, cw, offset=0):
    import torch

    import oracle
    import paper_1709_03708_amd as pq

    buf = torch.empty(vectors.size + offset, dtype=torch.float32, device="cuda")
    v = buf[offset:].view(vectors.shape)
    v.copy_(torch.from_numpy(vectors))
    got = pq.encode(v, torch.from_numpy(cw).cuda()).cpu().numpy()
    assert np.array_equal(got, oracle.encode(vectors, cw))


@pytest.mark.parametrize("Ds", [1, 2, 3, 4, 5, 6, 7, 8, 9, 16, 17])
@pytest.mark.parametrize("N,M", [(1, 1), (31, 9), (33, 8), (1025, 32), (20_011, 3)])
def test_lengths_and_tiles(Ds, N, M):
    rng = np.random.default_rng(Ds * 100_000 + N)
    cw = (20 * rng.standard_normal((M, 256, Ds)) + 3).astype(np.float32)
    vectors = (20 * rng.standard_normal((N, M * Ds)) + 3).astype(np.float32)
    _check(vectors, cw)
    _check(vectors, cw, 1)


@pytest.mark.parametrize("Ds", [3, 4, 7, 8])
def test_equal_lengths_and_ties(Ds):
    rng = np.random.default_rng(Ds)
    cw = rng.standard_normal((2, 256, Ds))
    cw = (cw / np.linalg.norm(cw, axis=2, keepdims=True)).astype(np.float32)
    for size in (1e-5, 1e-3, 1.0):
        _check((size * rng.standard_normal((500, 2 * Ds))).astype(np.float32), cw)
    cw[:, 128:] = cw[:, :128]                                          # the lower index wins
    vectors = rng.standard_normal((500, 2, Ds)).astype(np.float32)
    vectors[::3] = cw[:, 77]
    vectors[1::3] = 0.5 * (cw[:, 5] + cw[:, 6])
    _check(vectors.reshape(500, 2 * Ds), cw)


@pytest.mark.parametrize("Ds", [4, 6, 8])
@pytest.mark.parametrize("scale", [1e-42, 1e-30, 1e-19, 1e18, 3e37])
def test_scales_and_non_finite(Ds, scale):
    rng = np.random.default_rng(Ds)
    with np.errstate(over="ignore", under="ignore"):
        cw = (rng.standard_normal((3, 256, Ds)) * scale).astype(np.float32)
        vectors = (rng.standard_normal((300, 3 * Ds)) * scale).astype(np.float32)
        _check(vectors, cw)
        vectors[3, 1] = np.nan
        vectors[64, 2] = np.inf
        vectors[299] = -np.inf
        cw[1, 7, 3] = np.inf
        cw[2, 9] = np.nan
        _check(vectors, cw)
