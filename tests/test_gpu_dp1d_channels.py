"""RFSF-DP-1D at both edges of every number of channels that the kernel is compiled for."""
import math

import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from tests.parity import FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 18, 19, 24, 25, 32, 33, 40, 41, 48, 49, 64])
def test_channels(oracle, d):
    rng = np.random.default_rng(d)
    N, L, M, F = 5, 34, 3, 70                                # (fewer than 65 points: not the kernel of stretches)
    X = np.cumsum(rng.standard_normal((N, L, d)) / math.sqrt(L), axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    b = rng.uniform(0.0, 2.0 * math.pi, size=(M, F)).astype(np.float32)
    ls = float(np.float32(math.sqrt(d)))
    got = rfsf.rfsf_dp1d_features(*(torch.from_numpy(a).cuda() for a in (X, W, b)), ls).cpu().numpy()
    assert np.all(block_errors(got, oracle.dp1d_features(X, W, b, ls), M, F) <= FP32_BLOCK_TOL)
