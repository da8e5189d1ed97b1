"""Variable-length batches: the projection kernel leaves out tiles of rows that lie beyond the end of their sequence. The
last existing increment at every place around a tile's edges; sequences shorter than a tile; both operand types; NaN in
what the batch is padded with."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from tests.parity import BF16_BLOCK_TOL, FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,bf16", [(70, 333, False), (40, 640, False), (90, 20, False), (70, 334, True)])
def test_tiles_beyond_the_end(oracle, N, L, bf16):
    rng = np.random.default_rng(L)
    d, M, F, D = 3, 2, 20, 64
    X = np.cumsum(rng.standard_normal((N, L, d)) * 0.1, axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    hash_ = rng.integers(0, D, size=(M, 2 * F)).astype(np.int32)
    sign = (2.0 * rng.integers(0, 2, size=(M, 2 * F)) - 1.0).astype(np.float32)
    lengths = ((np.arange(N) * 37) % L + 1).astype(np.int64) if L < 100 else (1 + (np.arange(N) + L // 2) % L).astype(np.int64)
    padded = X.copy()
    for n in range(N):
        padded[n, lengths[n]:] = np.nan
    got = rfsf.rfsf_ts_features(torch.from_numpy(padded).cuda(), torch.from_numpy(W).cuda(), torch.from_numpy(hash_).cuda(),
                                torch.from_numpy(sign).cuda(), 1.5, D, rff_bf16=bf16,
                                lengths=torch.from_numpy(lengths).cuda()).cpu().numpy()
    err = block_errors(got, oracle.features_ragged(X, lengths, W, hash_, sign, 1.5, D), M, D)
    print(f"N={N} L={L} bf16={bf16}: block errors {err}")
    assert np.all(err <= (BF16_BLOCK_TOL if bf16 else FP32_BLOCK_TOL))
