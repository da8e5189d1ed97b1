"""Of `sign` only the sign bit is used (include/rfsf_ts.h), on every route of the features call: zeros and NaN of either sign are what
+1 and -1 with their sign bit are, bit for bit."""
import math

import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,d,M,F,D,bf16", [
    (300, 100, 8, 4, 128, 256, False),   # single wavefronts that compute their increments
    (100, 300, 5, 5, 50, 100, False),    # ... 100 points
    (3, 40, 5, 3, 20, 64, False),        # a workgroup per sequence
    (3, 40, 17, 4, 64, 256, False),      # projection on the matrix units
    (3, 40, 17, 4, 64, 256, True),       # ... of bf16 operands
    (3, 40, 66, 4, 64, 256, False),      # ... on the vector units
    (3, 40, 5, 9, 20, 64, False),        # generic consumer, row layout
])
def test_only_the_sign_bit_of_a_sign_counts(N, L, d, M, F, D, bf16):
    rng = np.random.default_rng(D + d)
    X = np.cumsum(rng.standard_normal((N, L, d)) * 0.2, axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    hash_ = rng.integers(0, D, size=(M, 2 * F)).astype(np.int32)
    plain = (2.0 * rng.integers(0, 2, size=(M, 2 * F)) - 1.0).astype(np.float32)
    other = np.copysign(rng.choice(np.array([0.0, 1.0, 3.0, 1e-42, math.inf, math.nan], dtype=np.float32), size=plain.shape), plain)
    X, W, hash_, plain, other = (torch.from_numpy(a).cuda() for a in (X, W, hash_, plain, other))
    want, got = (rfsf.rfsf_ts_features(X, W, hash_, s, math.sqrt(d), D, rff_bf16=bf16) for s in (plain, other))
    assert torch.equal(got, want)
