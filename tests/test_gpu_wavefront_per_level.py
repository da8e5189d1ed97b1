"""500 and 512 points with five and six levels: whole sequences of order 1 deal their items to eight wavefronts, those of orders 2 and 3 have a
wavefront per level. Iterations of two pairs: last ones with one and with two, odd and even numbers of steps; batches whose sequences are
taken by length. Tolerance: sine and cosine of 32-bit angles around 1 are off by 5e-8 (root mean square), a difference of two by
7e-8, increments are 0.13 in size (0.2 sqrt(5) / 2.5 / sqrt(2)): 5.5e-7 of an increment, sqrt(m) times that of a product of m, which
sums over steps only lower; times three."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,F,ragged", [(3, 2, 30, False), (3, 4, 30, True), (2, 13, 250, False), (2, 22, 700, False), (300, 60, 40, True)])
@pytest.mark.parametrize("M,order", [(5, 1), (5, 2), (5, 3), (6, 1), (6, 2), (6, 3)])
@pytest.mark.parametrize("D", [500, 512])
def test_whole_sequences_of_every_order(oracle, D, M, order, N, L, F, ragged):
    rng = np.random.default_rng(D + L + M)
    X = np.cumsum(rng.standard_normal((N, L, 5)) * 0.2, axis=1).astype(np.float32)
    W = rng.standard_normal((M, 5, F)).astype(np.float32)
    hash_ = rng.integers(0, D, size=(M, 2 * F)).astype(np.int32)
    sign = (2.0 * rng.integers(0, 2, size=(M, 2 * F)) - 1.0).astype(np.float32)
    lengths = rng.integers((L + 1) // 2, L + 1, size=N)
    on = [torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)]
    got = rfsf.rfsf_ts_features(*on, 2.5, D, order=order, lengths=torch.from_numpy(lengths).cuda() if ragged else None).cpu().numpy()
    rows = np.r_[0:N] if N < 10 else np.r_[0, 1, N // 2, N - 1]
    if ragged:
        want = oracle.features_ragged(X[rows], lengths[rows], W, hash_, sign, 2.5, D, order=order)
    else:
        want = oracle.features(X[rows], W, hash_, sign, 2.5, D, order=order)
    for m in range(M):
        g, w = (a[:, 1 + m * D:1 + (m + 1) * D].astype(np.float64) for a in (got[rows], want))
        assert np.linalg.norm(g - w) <= 1.65e-6 * np.sqrt(m + 1) * np.linalg.norm(w), m
