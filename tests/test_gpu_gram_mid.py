"""Gram products of 150 .. 256 tiles of 64 x 64, eight wavefronts each: both ends of the range and one tile beyond, columns
that leave wavefronts without a step or with a partial one, rows that are no multiple of anything, packed rows. Against 64
bits.

Tolerance. The errors of a sum of K products in 32 bits are independent roundings, and each of the products that are added
up in blocks of 32 columns is rounded into an accumulator at most about as large as the root of the sum of their squares
and the sum itself (which is the larger one on a diagonal), r = sqrt(sum a^2 b^2) + |sum a b|: a random walk of 1 + K / 32
steps of 2^-24 r. Eight times that, six standard deviations and what rounding downwards adds. The three terms of a number make six products; a kernel that leaves any of them out is outside
(checked below, on the CPU, on the same inputs)."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

SHAPES = [
    (640, 960, 65, 0), (640, 961, 65, 0),      # 150 and 160 tiles
    (1000, 1024, 1025, 3), (1024, 1024, 31, 0), (1024, 1025, 256, 0),
    (301, 2000, 257, 0),
    (1110, 0, 129, 3), (1400, 0, 513, 0),      # a batch with itself: 171 and 253 tiles
]


def _operands(Nx, Ny, K, pad):
    rng = np.random.default_rng(Nx + K)
    A = np.zeros((Nx, K + pad), dtype=np.float32)
    A[:, :K] = rng.standard_normal((Nx, K))
    B = A if Ny == 0 else rng.standard_normal((Ny, K)).astype(np.float32)
    return A, B


def _bound(A, B):
    a, b = A.astype(np.float64) ** 2, B.astype(np.float64) ** 2
    r = np.sqrt(a @ b.T) + np.abs(A.astype(np.float64) @ B.astype(np.float64).T)
    return 8 * np.sqrt(1 + A.shape[1] / 32) * 2.0 ** -24 * r


@pytest.mark.gpu
@pytest.mark.parametrize("Nx,Ny,K,pad", SHAPES)
def test_mid_products(Nx, Ny, K, pad):
    A, B = _operands(Nx, Ny, K, pad)
    a = torch.from_numpy(A).cuda()[:, :K]
    got = (rfsf.rfsf_ts_gram(a) if Ny == 0 else rfsf.rfsf_ts_gram(a, torch.from_numpy(B).cuda())).cpu().numpy()
    A, B = A[:, :K], B[:, :K]
    ratio = np.abs(got - A.astype(np.float64) @ B.astype(np.float64).T) / _bound(A, B)
    print(f"{Nx} x {Ny or Nx}, {K} columns: at most {ratio.max():.2f} of the bound")
    assert ratio.max() <= 1
    if Ny == 0:
        assert np.array_equal(got, got.T)


def _terms(x):
    """hi, mid and lo, each the bfloat16 next to what the ones before leave of x."""
    def nearest(v):
        u = v.astype(np.float32).view(np.uint32).astype(np.uint64)
        return ((u + 0x7fff + ((u >> 16) & 1)) >> 16 << 16).astype(np.uint32).view(np.float32)
    hi = nearest(x)
    mid = nearest(x - hi)
    return hi, mid, nearest(x - hi - mid)


@pytest.mark.parametrize("Nx,Ny,K,pad", SHAPES)
def test_bound_tells_a_missing_product(Nx, Ny, K, pad):
    A, B = _operands(Nx, Ny, K, pad)
    A, B = A[:400, :K], B[:400, :K]
    want, bound = A.astype(np.float64) @ B.astype(np.float64).T, _bound(A, B)
    ta, tb = [t.astype(np.float64) for t in _terms(A)], [t.astype(np.float64) for t in _terms(B)]
    assert np.array_equal(sum(ta), A) and np.array_equal(sum(tb), B)
    products = {(i, j): ta[i] @ tb[j].T for i in range(3) for j in range(3) if i + j <= 2}
    total = sum(products.values())
    assert (np.abs(total - want) / bound).max() <= 0.1           # the three products of the smallest terms
    for missing, p in products.items():
        assert (np.abs(total - p - want) / bound).max() > 1.5, missing
