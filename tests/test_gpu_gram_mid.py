"""Gram products of 150 .. 256 tiles of 64 x 64, eight wavefronts each: both ends of the range and one tile beyond, columns
that leave wavefronts without a step or with a partial one, rows that are no multiple of anything, packed rows. Against 64
bits; the tolerance is what sums of K products in 32 bits may differ by, K * 2^-24 of the largest |a| |b|, with a margin of 4."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Nx,Ny,K,pad", [
    (640, 960, 65, 0), (640, 961, 65, 0),      # 150 and 160 tiles
    (1000, 1024, 1025, 3), (1024, 1024, 31, 0), (1024, 1025, 256, 0),
    (301, 2000, 257, 0),
    (1110, 0, 129, 3), (1400, 0, 513, 0),      # a batch with itself: 171 and 253 tiles
])
def test_mid_products(Nx, Ny, K, pad):
    rng = np.random.default_rng(Nx + K)
    A = np.zeros((Nx, K + pad), dtype=np.float32)
    A[:, :K] = rng.standard_normal((Nx, K))
    B = A if Ny == 0 else rng.standard_normal((Ny, K)).astype(np.float32)
    a = torch.from_numpy(A).cuda()[:, :K]
    got = (rfsf.rfsf_ts_gram(a) if Ny == 0 else rfsf.rfsf_ts_gram(a, torch.from_numpy(B).cuda())).cpu().numpy()
    want = A[:, :K].astype(np.float64) @ B[:, :K].astype(np.float64).T
    bound = 4 * K * 2.0 ** -24 * np.linalg.norm(A[:, :K], axis=1).max() * np.linalg.norm(B[:, :K], axis=1).max()
    assert np.abs(got - want).max() <= bound
    if Ny == 0:
        assert np.array_equal(got, got.T)
