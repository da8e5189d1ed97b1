"""Transforms with more points than buckets: the linear route at the largest bucket counts that a length holds and just below, whose
empty groups of buckets are neither read nor transformed, and bucket counts that many features move to a longer transform, some of
which have too many groups for that. Tolerance: that of the butterflies' test (three times the error of 32-bit angles, sums and roots)."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,F,D,order", [
    (2, 40, 256 - 1, 1), (2, 40, 511, 1), (2, 40, 1023, 1),          # 512, 1024 and 2048 points, half of the groups
    (3, 40, 171, 1), (3, 40, 342, 1), (3, 40, 683, 1), (3, 40, 342, 3),
    (4, 40, 127, 1), (4, 40, 255, 2), (4, 40, 511, 1),               # a quarter
    (5, 40, 103, 1), (5, 40, 205, 1), (5, 40, 410, 2),
    (8, 40, 64 + 1, 1), (8, 200, 128 - 1, 1),
    (4, 1000, 64, 1), (4, 2000, 256, 1), (5, 2000, 512, 1),          # powers of two in longer transforms
    (7, 40, 146, 2), (7, 40, 146, 3), (7, 40, 292, 3),               # whole sequences whose middle pass has an exchange
    (4, 40, 1023, 3), (6, 40, 682, 3), (8, 40, 511, 1),              # ... and 4096 points
])
@pytest.mark.parametrize("L", [4, 23])
def test_empty_groups_of_buckets_are_left_out(oracle, M, F, D, order, L):
    rng = np.random.default_rng(D + L)
    X = np.cumsum(rng.standard_normal((3, L, 9)) * 0.2, axis=1).astype(np.float32)
    W = rng.standard_normal((M, 9, F)).astype(np.float32)
    hash_ = rng.integers(0, D, size=(M, 2 * F)).astype(np.int32)
    hash_[:, 0] = D - 1                                              # the last bucket is used
    sign = (2.0 * rng.integers(0, 2, size=(M, 2 * F)) - 1.0).astype(np.float32)
    got = rfsf.rfsf_ts_features(*(torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)), 3.0, D, order=order).cpu().numpy()
    want = oracle.features(X, W, hash_, sign, 3.0, D, order=order)
    for m in range(min(M, L - 1) if order == 1 else M):              # (no more steps than levels: blocks of zeros)
        g, w = (a[:, 1 + m * D:1 + (m + 1) * D].astype(np.float64) for a in (got, want))
        assert np.linalg.norm(g - w) <= 1.5e-6 * np.linalg.norm(w), m


@pytest.mark.parametrize("M,F,D,order", [
    (2, 60, 255, 2), (3, 60, 171, 1), (4, 60, 127, 2), (5, 60, 103, 1), (6, 60, 85, 3), (7, 60, 74, 2), (8, 60, 63, 1),      # 512 points
    (3, 200, 683, 2), (4, 200, 511, 1), (5, 200, 410, 2), (6, 200, 341, 3), (7, 200, 292, 1),                                # 2048
    (4, 120, 255, 2), (4, 120, 255, 3), (5, 120, 204, 1), (5, 120, 204, 2), (5, 120, 204, 3), (6, 120, 170, 2), (6, 120, 170, 3),      # 1024
])
def test_sequences_cut_in_time(oracle, M, F, D, order):
    """Pieces of a few sequences, whose kernels leave the empty groups out where that costs them no registers. Increments are 0.14 in size, of which
    32-bit angles, sines and cosines leave 7e-8 / 0.14, sqrt(m) times that of a product of m; three times that."""
    N, L = 2, 90
    rng = np.random.default_rng(D + M)
    X = np.cumsum(rng.standard_normal((N, L, 9)) * 0.2, axis=1).astype(np.float32)
    W = rng.standard_normal((M, 9, F)).astype(np.float32)
    hash_ = rng.integers(0, D, size=(M, 2 * F)).astype(np.int32)
    hash_[:, 0] = D - 1
    sign = (2.0 * rng.integers(0, 2, size=(M, 2 * F)) - 1.0).astype(np.float32)
    got = rfsf.rfsf_ts_features(*(torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)), 3.0, D, order=order).cpu().numpy()
    want = oracle.features(X, W, hash_, sign, 3.0, D, order=order)
    for m in range(M):
        g, w = (a[:, 1 + m * D:1 + (m + 1) * D].astype(np.float64) for a in (got, want))
        assert np.linalg.norm(g - w) <= 1.5e-6 * np.sqrt(m + 1) * np.linalg.norm(w), m
