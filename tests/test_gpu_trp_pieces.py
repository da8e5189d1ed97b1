"""RFSF-TRP of few long sequences: the recurrence runs on pieces whose sums take the place of the projected increments,
and the pieces are joined. Lengths at which the last piece is short or the only cut possible is the smallest."""
import math

import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from tests.parity import FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,M,Q", [
    (1, 129, 3, 20),            # four pieces of 32 steps, the shortest sequence that is cut
    (1, 128, 3, 20),            # one step less: whole
    (3, 1058, 8, 16),           # 33 pieces would leave the last too short for the sums of eight levels
    (2, 1059, 8, 7),
    (2, 4001, 1, 33),
    (5, 700, 5, 200),
    (2, 500, 9, 12),            # nine levels: whole
    (2, 9000, 4, 64),
])
def test_pieces_match_the_oracle(oracle, N, L, M, Q):
    rng = np.random.default_rng(L + Q)
    d, F = 3, 12
    X = np.cumsum(rng.standard_normal((N, L, d)) * 0.1, axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    Z = rng.standard_normal((M, Q, 2 * F)).astype(np.float32)
    ls = float(np.float32(math.sqrt(d)))
    got = rfsf.rfsf_trp_features(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), torch.from_numpy(Z).cuda(), ls)
    err = block_errors(got.cpu().numpy(), oracle.trp_features(X, W, Z, ls), M, Q)
    print(f"N={N} L={L} M={M} Q={Q}: block errors {err}")
    assert np.all(err <= FP32_BLOCK_TOL)


@pytest.mark.parametrize("N,L,M,Q", [(1, 2000, 5, 33), (3, 700, 4, 50)])
def test_pieces_of_noise(oracle, N, L, M, Q):
    """Increments that do not get smaller with the number of points: what the pieces add up cancels."""
    rng = np.random.default_rng(L + Q)
    d, F = 1, 64
    X = rng.standard_normal((N, L, d)).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    Z = rng.standard_normal((M, Q, 2 * F)).astype(np.float32)
    got = rfsf.rfsf_trp_features(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), torch.from_numpy(Z).cuda(), 1.0)
    err = block_errors(got.cpu().numpy(), oracle.trp_features(X, W, Z, 1.0), M, Q)
    print(f"noise N={N} L={L} M={M} Q={Q}: block errors {err}")
    assert np.all(err <= FP32_BLOCK_TOL)
