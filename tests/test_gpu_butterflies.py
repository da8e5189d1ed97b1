"""Transforms of every length and radix against the oracle, closely enough that a single wrong twiddle or root shows: error of a
level over its numbers, 2-norms. Angles and cosines in 32 bits leave 2e-7 to 3e-7 of the first level and 1e-7 more per level
(measured, all lengths); a twiddle off by 1e-6 in one of the ten stages would add as much. The bound is three times the largest."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,F,D", [
    (2, 24, 48),                                             # folded from 64 or 128 points
    (3, 32, 64), (3, 64, 128), (3, 128, 256), (3, 256, 512), (3, 512, 1024), (2, 512, 2048),
    (3, 50, 100), (3, 100, 200), (3, 250, 500), (3, 300, 1000),
    (3, 100, 1300), (3, 100, 2500),                          # 4096 and 8192 points
])
@pytest.mark.parametrize("L", [8, 19])                       # odd and even numbers of steps
def test_transforms_match_the_oracle(oracle, M, F, D, L):
    rng = np.random.default_rng(D + L)
    X = np.cumsum(rng.standard_normal((3, L, 9)) * 0.2, axis=1).astype(np.float32)
    W = rng.standard_normal((M, 9, F)).astype(np.float32)
    hash_ = rng.integers(0, D, size=(M, 2 * F)).astype(np.int32)
    sign = (2.0 * rng.integers(0, 2, size=(M, 2 * F)) - 1.0).astype(np.float32)
    got = rfsf.rfsf_ts_features(*(torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)), 3.0, D).cpu().numpy()
    want = oracle.features(X, W, hash_, sign, 3.0, D)
    for m in range(M):
        g, w = (a[:, 1 + m * D:1 + (m + 1) * D].astype(np.float64) for a in (got, want))
        error = np.linalg.norm(g - w) / np.linalg.norm(w)
        assert error <= 1.5e-6, (m, error)
