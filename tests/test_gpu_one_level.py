"""One level: the increments of a sequence are added up before the only transform. No, one, two and three steps, odd and
even numbers of them, lengths of their own, split sequences and whole ones, every family of transforms."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from tests.parity import FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,F,D,order", [
    (3, 2, 16, 64, 1), (3, 3, 16, 64, 1), (3, 4, 33, 64, 2),
    (300, 21, 50, 100, 1),         # whole sequences
    (300, 22, 200, 64, 1),
    (2, 500, 70, 256, 1),          # split
    (2, 131, 40, 200, 3),
    (5, 40, 600, 512, 1),
    (4, 61, 30, 1024, 1), (4, 62, 300, 1000, 2), (3, 64, 500, 2048, 1),
    (2, 30, 20, 300, 1), (2, 30, 20, 4096, 1),
])
def test_one_level(oracle, N, L, F, D, order):
    rng = np.random.default_rng(N + L + D)
    d = 3
    X = np.cumsum(rng.standard_normal((N, L, d)) * 0.2, axis=1).astype(np.float32)
    W = rng.standard_normal((1, d, F)).astype(np.float32)
    hash_ = rng.integers(0, D, size=(1, 2 * F)).astype(np.int32)
    sign = (2.0 * rng.integers(0, 2, size=(1, 2 * F)) - 1.0).astype(np.float32)
    lengths = np.where(rng.random(N) < 0.4, L, rng.integers(1, L + 1, size=N)).astype(np.int64)
    for own in (None, lengths):
        got = rfsf.rfsf_ts_features(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), torch.from_numpy(hash_).cuda(),
                                    torch.from_numpy(sign).cuda(), 1.5, D, order=order,
                                    lengths=None if own is None else torch.from_numpy(own).cuda()).cpu().numpy()
        want = oracle.features_ragged(X, np.full(N, L, dtype=np.int64) if own is None else own, W, hash_, sign, 1.5, D,
                                      order=order)
        err = block_errors(got, want, 1, D)
        print(f"N={N} L={L} F={F} D={D} order {order}: block errors {err}")
        assert np.all(err <= FP32_BLOCK_TOL)
