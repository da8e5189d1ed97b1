"""RFSF-DP-1D of few sequences: a workgroup's wavefronts share out the time points and their sums are joined. Lengths at
which the stretches come out whole, one step longer, or run out before the last wavefront."""
import math

import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from tests.parity import FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,d,M,F", [
    (1, 64, 3, 5, 70),           # one point too short: whole
    (1, 65, 3, 5, 70),           # three stretches of 31, 31 and 2 steps
    (1, 249, 3, 5, 70),          # eight stretches of one tile
    (1, 250, 3, 4, 64),          # one step more: four of two tiles
    (2, 250, 17, 4, 130),
    (3, 700, 32, 5, 65),
    (2, 300, 60, 4, 33),
    (2, 300, 60, 5, 33),         # too many channels and levels: whole
    (1, 100, 2, 1, 5),
    (128, 70, 5, 2, 256),        # the largest batch that is shared out
    (129, 70, 5, 2, 256),        # the smallest that is not
])
def test_stretches_match_the_oracle(oracle, N, L, d, M, F):
    rng = np.random.default_rng(L + F)
    X = np.cumsum(rng.standard_normal((N, L, d)) * 0.1, axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    bias = (rng.random((M, F)) * 2 * np.pi).astype(np.float32)
    ls = float(np.float32(math.sqrt(d)))
    got = rfsf.rfsf_dp1d_features(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), torch.from_numpy(bias).cuda(), ls)
    err = block_errors(got.cpu().numpy(), oracle.dp1d_features(X, W, bias, ls), M, F)
    print(f"N={N} L={L} d={d} M={M} F={F}: block errors {err}")
    assert np.all(err <= FP32_BLOCK_TOL)


@pytest.mark.parametrize("N,L,M,F", [(1, 2000, 5, 64), (3, 700, 4, 130)])
def test_stretches_of_noise(oracle, N, L, M, F):
    rng = np.random.default_rng(L + F)
    X = rng.standard_normal((N, L, 1)).astype(np.float32)
    W = rng.standard_normal((M, 1, F)).astype(np.float32)
    bias = (rng.random((M, F)) * 2 * np.pi).astype(np.float32)
    got = rfsf.rfsf_dp1d_features(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), torch.from_numpy(bias).cuda(), 1.0)
    err = block_errors(got.cpu().numpy(), oracle.dp1d_features(X, W, bias, 1.0), M, F)
    print(f"noise N={N} L={L} M={M} F={F}: block errors {err}")
    assert np.all(err <= FP32_BLOCK_TOL)
