"""Parity of the overlap histogram (int8 MFMA pair products) with the oracle:
bit-exact integer counts, including ragged batches and spin counts, the
all-configurations closed form, and exact first and second moments at the
benchmark size (16384 samples of 1000 spins)."""
import math

import numpy as np
import pytest
import torch

import paper_2606_22984_amd as fv
from oracle import overlap, physics
from tests.gpu_util import say, to_np
from workloads.instances import random_spins

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N", [(1, 5), (2, 7), (64, 100), (65, 1000), (200, 33), (130, 64), (77, 16000)])
def test_overlap_histogram_matches_oracle(B, N):
    s = random_spins(B, N, B * 31 + N)
    say(f"overlap B={B} N={N}")
    got = to_np(fv.overlap_histogram(torch.as_tensor(s, device="cuda")))
    assert np.array_equal(got, overlap.overlap_counts(s))


def test_overlap_histogram_all_configurations():
    n = 12
    got = to_np(fv.overlap_histogram(torch.as_tensor(physics.all_configs(n), device="cuda")))
    assert got.tolist() == [2 ** (n - 1) * math.comb(n, k) for k in range(n)] + [0]


def test_overlap_histogram_moments_at_benchmark_size():
    B, N = 16384, 1000
    rng = np.random.default_rng(5)
    s = np.where(rng.random((B, N)) < 0.45, -1, 1).astype(np.int8)
    got = to_np(fv.overlap_histogram(torch.as_tensor(s, device="cuda"))).astype(np.int64)
    x = 2 * np.arange(N + 1, dtype=np.int64) - N        # s_a . s_b of each bin
    assert got.sum() == B * (B - 1) // 2
    col = s.astype(np.int64).sum(axis=0)
    m1 = (int((col * col).sum()) - B * N) // 2             # sum over a < b of s_a . s_b
    assert int((got * x).sum()) == m1
    f = s.astype(np.float64)
    G = f.T @ f                                            # exact: integer entries <= B
    m2 = (int(np.rint((G * G).sum())) - B * N * N) // 2    # sum over a < b of (s_a . s_b)^2
    assert int((got * x * x).sum()) == m2


@pytest.mark.parametrize("B,N,start", [(64, 64, 0), (63, 1, 3), (3968, 65, 0), (3969, 63, 1), (4033, 130, 5),
                                       (7937, 70, 0), (8065, 1023, 2), (8000, 1024, 0), (300, 9000, 0)])
def test_overlap_histogram_block_edges(B, N, start):
    """Exact counts at the edges of the three block sizes and of the histogram copies, with ragged rows and a
    batch that starts `start` bytes into its allocation.  The counts are those of the integer product S S^T."""
    rng = np.random.default_rng(B + N)
    s = np.where(rng.random((B, N)) < 0.3, -1, 1).astype(np.int8)
    store = torch.zeros(B * N + start, dtype=torch.int8, device="cuda")
    store[start:] = torch.as_tensor(s.reshape(-1), device="cuda")
    say(f"overlap B={B} N={N} start={start}")
    got = to_np(fv.overlap_histogram(store[start:].view(B, N)))
    f = s.astype(np.float32)
    ref = np.zeros(N + 1, dtype=np.int64)
    for a in range(0, B, 1024):                    # integers below 2^24: exact in float32
        q = f[a:a + 1024] @ f.T
        k = ((q + N) / 2).astype(np.int64)
        upper = np.arange(B)[None, :] > np.arange(a, min(a + 1024, B))[:, None]
        ref += np.bincount(k[upper], minlength=N + 1)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("B,N", [(1408, 66), (1409, 66), (1856, 130), (1857, 130), (1500, 14001), (3968, 300), (6000, 64),
                                 (6000, 65), (7100, 64)])
def test_overlap_histogram_where_the_block_size_changes(B, N):
    """Exact counts on both sides of the rule's lines between blocks of 64, 128 and 256 samples (one and two block
    pairs of 64 per compute unit, one to three rounds of the larger ones, histograms too large for two)."""
    g = torch.Generator(device="cuda").manual_seed(B + N)
    s = torch.randint(0, 2, (B, N), generator=g, device="cuda", dtype=torch.int8) * 2 - 1
    say(f"overlap B={B} N={N}")
    got = to_np(fv.overlap_histogram(s))
    f = to_np(s).astype(np.float32)
    ref = np.zeros(N + 1, dtype=np.int64)
    for a in range(0, B, 1024):                    # integers below 2^24: exact in float32
        k = ((f[a:a + 1024] @ f.T + N) / 2).astype(np.int64)
        upper = np.arange(B)[None, :] > np.arange(a, min(a + 1024, B))[:, None]
        ref += np.bincount(k[upper], minlength=N + 1)
    assert np.array_equal(got, ref)
