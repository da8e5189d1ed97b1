"""RFSF-DP-1D with frequencies resident in LDS: every number of channels that the kernel is compiled for, at both edges; last tiles of
one row, of whole groups of eight and one more; blocks of components that are not full; more sequences than wavefronts, and fewer."""
import math

import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from tests.parity import FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


def _case(N, L, d, M, F):
    rng = np.random.default_rng(N + L + d + F)
    X = np.cumsum(rng.standard_normal((N, L, d)) / math.sqrt(L), axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    b = rng.uniform(0.0, 2.0 * math.pi, size=(M, F)).astype(np.float32)
    return X, W, b, float(np.float32(math.sqrt(d)))


@pytest.mark.parametrize("N,L,d,M,F", [
    (200, 33, d, 3, 70) for d in (1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 18, 19, 24, 25, 32, 33, 40, 41, 48, 49, 64)
] + [
    (300, 1, 17, 2, 64), (300, 2, 17, 5, 65), (300, 8, 9, 4, 128), (300, 9, 9, 4, 129), (300, 31, 12, 3, 200), (300, 32, 12, 3, 200),
    (300, 57, 17, 5, 1000), (300, 96, 20, 4, 63), (4000, 40, 17, 5, 64), (3100, 5, 30, 2, 300), (700, 70, 10, 16, 40), (150, 66, 64, 5, 130),
    (150, 66, 64, 6, 130), (129, 70, 5, 2, 256),
])
def test_rows_match_the_oracle(oracle, N, L, d, M, F):
    X, W, b, ls = _case(N, L, d, M, F)
    dev = [torch.from_numpy(a).cuda() for a in (X, W, b)]
    got = rfsf.rfsf_dp1d_features(*dev, ls)
    assert torch.equal(got, rfsf.rfsf_dp1d_features(*dev, ls))
    rows = np.unique(np.array([0, 1, N // 2, N - 2, N - 1]))
    err = block_errors(got.cpu().numpy()[rows], oracle.dp1d_features(X[rows], W, b, ls), M, F)
    assert np.all(err <= FP32_BLOCK_TOL), err


def test_nan_and_infinity_stay_where_they_are():
    N, L, d, M, F = 300, 40, 17, 3, 130
    X, W, b, ls = _case(N, L, d, M, F)
    dev = [torch.from_numpy(a).cuda() for a in (X, W, b)]
    want = rfsf.rfsf_dp1d_features(*dev, ls)
    dev[0][7, 20, 3] = float("nan")
    dev[0][9, 39, 16] = float("inf")
    dev[1][1, 4, 77] = float("nan")
    dev[1][2, 0, 5] = float("-inf")
    got = rfsf.rfsf_dp1d_features(*dev, ls)
    bad = torch.zeros_like(want, dtype=torch.bool)
    bad[[7, 9], 1:] = True
    bad[:, 1 + F + 77] = bad[:, 1 + 2 * F + 77] = True       # a level and those above it
    bad[:, 1 + 2 * F + 5] = True
    assert bool(torch.isnan(got[bad]).all()) and torch.equal(got[~bad], want[~bad])


def test_sums_of_products_are_as_good_as_in_32_bits():
    """Phase 0 and one increment from the origin: level 1 is sqrt(2 / F) (cos(x . w) - 1). An angle is the sum of eight sums that
    each round once, by 2^-23 of the largest one at most, and is rounded to half-turns, 2^-24 with the rounding of their number in
    a radian; the cosine adds 2e-7. Root mean square 1.5e-6: a tenth of that bound for the mean angle; operands of 16 bits give 1e-2. Nor is it
    larger than what products added one after another in 32 bits give, rounded once each, with an exact cosine of half-turns in 32 bits (1.1e-6)."""
    rng = np.random.default_rng(5)
    N, d, F = 400, 17, 256
    X = np.zeros((N, 2, d), np.float32)
    X[:, 1] = rng.standard_normal((N, d)) * 3.0
    W = rng.standard_normal((1, d, F)).astype(np.float32)
    got = rfsf.rfsf_dp1d_features(*(torch.from_numpy(a).cuda() for a in (X, W, np.zeros((1, F), np.float32))), 1.0).cpu().numpy()
    angle = X[:, 1].astype(np.float64) @ W[0].astype(np.float64)
    err = got[:, 1:].astype(np.float64) * math.sqrt(F) - math.sqrt(2.0) * (np.cos(angle) - 1.0)
    bound = math.sqrt(2.0) * np.abs(angle).max() * (8 * 2.0 ** -23 + 2.0 ** -24) + 2e-7
    assert np.abs(err).max() <= bound and np.sqrt(np.mean(err ** 2)) <= 1.5e-6, (np.abs(err).max(), np.sqrt(np.mean(err ** 2)))
    sums = np.zeros((N, F), np.float32)
    for c in range(d):
        sums = (sums + np.outer(X[:, 1, c].astype(np.float64), W[0, c])).astype(np.float32)
    err_32 = math.sqrt(2.0) * (np.cos((sums * np.float32(1.0 / math.pi)).astype(np.float64) * math.pi) - np.cos(angle))
    assert np.sqrt(np.mean(err ** 2)) <= np.sqrt(np.mean(err_32 ** 2)), (np.sqrt(np.mean(err ** 2)), np.sqrt(np.mean(err_32 ** 2)))


@pytest.mark.parametrize("x,w,scale", [(-120, 0, -120), (-125, 125, 0), (-110, 70, -40), (100, -100, 0), (-20, -105, -126), (-62, 62, 0), (-66, 66, 0)])
def test_small_numbers_keep_their_bits(x, w, scale):
    """The same angles from points of 2^x and frequencies of 2^w over a lengthscale of 2^scale: powers of two change no bit of a
    32-bit product, so the bound of the test above holds. Points whose last 16-bit
    term would be lost (1e-4 and more) are raised before they are split."""
    assert x + w in (scale, scale + 1)
    rng = np.random.default_rng(6)
    N, d, F = 400, 17, 256
    X = np.zeros((N, 2, d), np.float32)
    X[:, 1] = rng.standard_normal((N, d)) * 2.0 ** x
    W = (rng.standard_normal((1, d, F)) * 2.0 ** w).astype(np.float32)
    got = rfsf.rfsf_dp1d_features(*(torch.from_numpy(a).cuda() for a in (X, W, np.zeros((1, F), np.float32))), 2.0 ** scale).cpu().numpy()
    angle = (X[:, 1].astype(np.float64) @ W[0].astype(np.float64)) / 2.0 ** scale
    err = got[:, 1:].astype(np.float64) * math.sqrt(F) - math.sqrt(2.0) * (np.cos(angle) - 1.0)
    assert np.sqrt(np.mean(err ** 2)) <= 1.5e-6, np.sqrt(np.mean(err ** 2))


@pytest.mark.parametrize("large", ["points", "frequencies"])
def test_largest_numbers_stay_finite(large):
    """Numbers within 2^-8 of the largest 32-bit one, beyond the largest of 16 bits, which a first term must not round up to; the others
    are small, so that the angles are of a few radians as above, with the bound of the test of sums."""
    rng = np.random.default_rng(7)
    N, d, F = 400, 17, 256
    X = np.zeros((N, 2, d), np.float32)
    X[:, 1] = rng.standard_normal((N, d))
    W = rng.standard_normal((1, d, F)).astype(np.float32)
    a, b = (X[:, 1], W) if large == "points" else (W, X[:, 1])
    a[...] = np.float32(np.finfo(np.float32).max) * rng.uniform(1.0 - 2.0 ** -9, 1.0, a.shape).astype(np.float32) * rng.choice((-1.0, 1.0), a.shape).astype(np.float32)
    b[...] *= 2.0 ** -60
    scale = 2.0 ** 67
    got = rfsf.rfsf_dp1d_features(*(torch.from_numpy(a).cuda() for a in (X, W, np.zeros((1, F), np.float32))), scale).cpu().numpy()
    angle = (X[:, 1].astype(np.float64) @ W[0].astype(np.float64)) / scale
    err = got[:, 1:].astype(np.float64) * math.sqrt(F) - math.sqrt(2.0) * (np.cos(angle) - 1.0)
    assert np.sqrt(np.mean(err ** 2)) <= 1.5e-6, np.sqrt(np.mean(err ** 2))


@pytest.mark.parametrize("N,L,d,M,F", [
    (N, L, d, M, 130) for N in (1, 2, 13) for L, d, M in ((2, 17, 3), (33, 7, 2), (64, 40, 5), (100, 12, 6))         # mostly idle workgroups
] + [
    (1, 8, 9, 1, 60), (1, 9, 9, 1, 60), (256, 20, 9, 1, 60), (257, 20, 9, 1, 60), (512, 20, 5, 1, 60), (513, 20, 5, 1, 60),         # one level
    (256, 5, 33, 1, 60), (257, 5, 33, 1, 60), (300, 33, 18, 1, 400), (300, 33, 18, 1, 500), (700, 64, 50, 1, 180), (700, 64, 50, 1, 250),
    (60, 18, 60, 2, 1010), (500, 32, 6, 2, 190), (500, 32, 6, 2, 250),
])
def test_small_batches_and_few_levels(oracle, N, L, d, M, F):
    """Sizes on both sides of the lines between this kernel and the one for one workgroup per sequence, which small batches of one level and
    a few points take."""
    X, W, b, ls = _case(N, L, d, M, F)
    got = rfsf.rfsf_dp1d_features(*(torch.from_numpy(a).cuda() for a in (X, W, b)), ls).cpu().numpy()
    rows = np.unique(np.array([0, N // 2, N - 1]))
    err = block_errors(got[rows], oracle.dp1d_features(X[rows], W, b, ls), M, F)
    assert np.all(err <= FP32_BLOCK_TOL), err
