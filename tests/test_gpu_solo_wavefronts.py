"""Short transforms whose levels fit one wavefront: whole sequences and pieces, increments computed in the kernel or read from
memory, at the edges of its rules (levels, channels, frequencies per lane, sequences of half an iteration and of one more
pair than an iteration, the smallest batch that takes it, pieces, points beyond a sequence's end)."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from tests.parity import FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


def _case(seed, N, L, d, M, F, D):
    rng = np.random.default_rng(seed)
    X = np.cumsum(rng.standard_normal((N, L, d)) * 0.2, axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    hash_ = rng.integers(0, D, size=(M, 2 * F)).astype(np.int32)
    sign = (2.0 * rng.integers(0, 2, size=(M, 2 * F)) - 1.0).astype(np.float32)
    return X, W, hash_, sign


@pytest.mark.parametrize("N,L,d,M,F,D", [
    (257, 33, 1, 2, 64, 64), (300, 20, 2, 3, 33, 64), (300, 17, 3, 4, 64, 64), (300, 26, 4, 5, 17, 64),
    (257, 49, 5, 2, 50, 100), (300, 50, 6, 3, 64, 100), (300, 25, 7, 4, 50, 100), (300, 18, 8, 5, 50, 100), (300, 19, 3, 6, 40, 100),
    (300, 34, 9, 5, 50, 100), (300, 34, 3, 5, 65, 100), (300, 34, 3, 5, 100, 100),          # increments from memory
    (300, 130, 3, 2, 64, 128), (300, 67, 1, 3, 30, 128), (300, 66, 8, 4, 64, 128),
    (300, 100, 5, 2, 100, 200), (300, 67, 2, 3, 128, 200), (300, 35, 4, 5, 65, 200),
    (300, 66, 8, 2, 32, 256), (300, 34, 3, 3, 64, 256), (300, 65, 8, 4, 128, 256), (300, 66, 3, 4, 97, 256),
    (100, 300, 5, 5, 50, 100), (100, 301, 2, 3, 30, 64), (90, 200, 8, 4, 128, 256),          # split
    (10, 2000, 5, 5, 50, 100), (60, 400, 3, 3, 64, 128),                                      # cut by the reported plan
    (2000, 10, 2, 5, 50, 100), (1100, 40, 2, 4, 30, 64),
])
def test_rows_match_the_oracle(oracle, N, L, d, M, F, D):
    X, W, hash_, sign = _case(N + L + D + d, N, L, d, M, F, D)
    rng = np.random.default_rng(L)
    rows = np.unique(rng.integers(0, N, size=8))
    dev = [torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)]
    for lengths in (None, np.where(rng.random(N) < 0.3, L, rng.integers(1, L + 1, size=N)).astype(np.int64)):
        kw = {}
        if lengths is not None:
            kw["lengths"] = torch.from_numpy(lengths).cuda()
            dev[0] = dev[0].clone()
            for n in rows:                 # what lies beyond a sequence's end is not read
                dev[0][n, lengths[n]:] = float("nan")
        got = rfsf.rfsf_ts_features(*dev, 1.5, D, **kw)
        again = rfsf.rfsf_ts_features(*dev, 1.5, D, **kw)
        assert torch.equal(got, again)
        for n in rows:
            x = X[n:n + 1] if lengths is None else X[n:n + 1, :lengths[n]]
            want = oracle.features(x, W, hash_, sign, 1.5, D)
            err = block_errors(got[int(n):int(n) + 1].cpu().numpy(), want, M, D)
            assert np.all(err <= FP32_BLOCK_TOL), (n, err)


@pytest.mark.parametrize("N,L,d,M,F,D,solo", [
    (600, 20, 8, 3, 20, 100, False), (600, 20, 4, 3, 20, 100, True),        # few frequencies per channel
    (600, 20, 12, 3, 60, 100, False), (600, 20, 12, 5, 60, 100, True),      # increments from memory
    (600, 18, 8, 4, 20, 64, False), (600, 18, 12, 4, 20, 64, False), (600, 18, 3, 4, 20, 64, True),
])
def test_short_sequences_that_gain_nothing(N, L, d, M, F, D, solo):
    """The kernel with a wavefront per level runs a single sequence of so few points whole, and sums it in another order."""
    X, W, hash_, sign = _case(N + F, N, L, d, M, F, D)
    dev = [torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)]
    one = rfsf.rfsf_ts_features(dev[0][5:6].contiguous(), *dev[1:], 1.5, D)
    assert torch.equal(rfsf.rfsf_ts_features(*dev, 1.5, D)[5:6], one) != solo


@pytest.mark.parametrize("N,L,M,F,D", [(600, 40, 3, 32, 64), (600, 40, 5, 50, 100), (600, 66, 3, 64, 256)])
def test_large_angles_are_as_accurate_as_the_products(oracle, N, L, M, F, D):
    """Products of points and frequencies that are exact in 32 bits, angles of some hundred: what is left are the errors of sine and
    cosine (6e-8) and of transforms and sums, 1e-7 to 3e-7 per level as for small angles. An angle rounded to 32 bits is off by
    up to 2^-24 of itself, 1e-5 and more."""
    rng = np.random.default_rng(D)
    X = (rng.integers(-2000, 2000, size=(N, L, 1)) / 8.0).astype(np.float32)
    W = (2.0 ** rng.integers(-2, 3, size=(M, 1, F)) * rng.choice((-1.0, 1.0), size=(M, 1, F))).astype(np.float32)
    _, _, hash_, sign = _case(D, 1, 2, 1, M, F, D)
    got = rfsf.rfsf_ts_features(*(torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)), 1.5, D).cpu().numpy()
    sel = [0, 5, N - 1]
    want = np.asarray(oracle.features(X[sel], W, hash_, sign, 1.5, D), np.float64)
    for m in range(1, M):                                    # (level 1 is a difference of two features, small against its sums)
        a, b = got[sel, 1 + m * D:1 + (m + 1) * D], want[:, 1 + m * D:1 + (m + 1) * D]
        assert np.linalg.norm(a - b) <= 3e-6 * np.linalg.norm(b), (m, np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("N,L,d,M,F,D", [
    (100, 1000, 5, 5, 50, 100), (300, 301, 2, 5, 50, 100), (420, 85, 3, 4, 60, 64), (350, 277, 2, 4, 64, 128), (500, 150, 7, 4, 41, 128),
    (700, 131, 8, 4, 100, 256), (300, 120, 8, 2, 64, 64), (300, 120, 4, 2, 39, 100),
    (60, 200, 8, 4, 50, 100), (60, 200, 8, 3, 50, 100), (50, 120, 8, 3, 60, 128), (40, 129, 8, 4, 128, 256),      # one to a CU just so
    (51, 200, 8, 5, 50, 100), (52, 200, 8, 5, 50, 100), (64, 81, 8, 3, 64, 256), (65, 81, 8, 3, 64, 256),
    (38, 200, 8, 5, 50, 100), (39, 200, 8, 5, 50, 100), (51, 81, 8, 3, 64, 256), (52, 81, 8, 3, 64, 256),         # both sides of the line
    (59, 172, 3, 5, 47, 64), (47, 184, 3, 5, 20, 64), (43, 118, 7, 4, 58, 128),                                    # one iteration each
])
def test_pieces_of_a_wavefronts_pairs(oracle, N, L, d, M, F, D):
    """Pieces of whole numbers of a wavefront's pairs and no whole number of iterations, so that the last wavefronts have less to do
    or nothing; slots of all distances; points in vector and in scalar registers."""
    X, W, hash_, sign = _case(N + L + D, N, L, d, M, F, D)
    got = rfsf.rfsf_ts_features(*(torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)), 1.5, D).cpu().numpy()
    for n in (0, 7, N - 1):
        err = block_errors(got[n:n + 1], oracle.features(X[n:n + 1], W, hash_, sign, 1.5, D), M, D)
        assert np.all(err <= FP32_BLOCK_TOL), (n, err)


@pytest.mark.parametrize("bits", [22, 23, 24])
def test_angles_of_millions(oracle, bits):
    """Angles of up to 2^bits radians from exact products, that is, on both sides of 2^22 quarter-turns and up to 2^23.3 of them. The
    number of quarter-turns in a unit is held to 2^-48 of itself: 2^-25 of a quarter-turn at 2^23 of them, which is what the
    reduced argument is rounded to as well. A single sequence, whose increments another kernel computes, has the same features."""
    N, L, M, F, D = 600, 40, 3, 32, 64
    rng = np.random.default_rng(4)
    X = rng.integers(-2 ** 20, 2 ** 20, size=(N, L, 1)).astype(np.float32)
    W = (2.0 ** rng.integers(bits - 25, bits - 19, size=(M, 1, F)) * rng.choice((-1.0, 1.0), size=(M, 1, F))).astype(np.float32)
    _, _, hash_, sign = _case(D, 1, 2, 1, M, F, D)
    dev = [torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)]
    got = rfsf.rfsf_ts_features(*dev, 1.0, D).cpu().numpy()
    for n in (0, 5, N - 1):
        want = oracle.features(X[n:n + 1], W, hash_, sign, 1.0, D)
        one = rfsf.rfsf_ts_features(dev[0][n:n + 1].contiguous(), *dev[1:], 1.0, D).cpu().numpy()
        for row in (got[n:n + 1], one):
            err = block_errors(row, want, M, D)
            assert np.all(err <= FP32_BLOCK_TOL), (n, err)


def test_chunks_and_bf16_projection_take_the_same_sums(oracle):
    """The cut is a function of the shape: a workspace for a part of the batch gives the same bits."""
    X, W, hash_, sign = _case(1, 600, 60, 5, 5, 50, 100)
    dev = [torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)]
    for bf16 in (False, True):
        rec, least = rfsf.rfsf_ts_workspace_bytes(600, 60, 5, 5, 50, 100, bf16)
        per = (rec - least) // 599
        whole = rfsf.rfsf_ts_features(*dev, 1.5, 100, rff_bf16=bf16)
        part = rfsf.rfsf_ts_features(*dev, 1.5, 100, rff_bf16=bf16,
                                     workspace=torch.empty(least + 250 * per, dtype=torch.uint8, device="cuda"))
        assert torch.equal(whole, part)


def test_nan_stays_in_its_sequence():
    X, W, hash_, sign = _case(2, 300, 40, 4, 4, 30, 64)
    dev = [torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)]
    want = rfsf.rfsf_ts_features(*dev, 1.5, 64)
    dev[0][7, 20, 1] = float("nan")
    dev[0][9, 3, 0] = float("inf")
    got = rfsf.rfsf_ts_features(*dev, 1.5, 64)
    bad = torch.zeros(300, dtype=torch.bool, device="cuda")
    bad[[7, 9]] = True
    assert bool(torch.isnan(got[bad][:, 1:]).all()) and torch.equal(got[~bad], want[~bad])


@pytest.mark.parametrize("d,projections", [(5, 0), (12, 3)])
def test_profile_counts_what_is_launched(d, projections):
    """Three launches of a batch: no projection where the sketch kernel does it, and one launch more for its tables."""
    X, W, hash_, sign = _case(3, 600, 60, d, 5, 50, 100)
    dev = [torch.from_numpy(a).cuda() for a in (X, W, hash_, sign)]
    rec, least = rfsf.rfsf_ts_workspace_bytes(600, 60, d, 5, 50, 100)
    ws = torch.empty(least + 250 * ((rec - least) // 599), dtype=torch.uint8, device="cuda")
    rfsf.rfsf_ts_profile_enable(True)
    rfsf.rfsf_ts_profile_read(True)
    rfsf.rfsf_ts_features(*dev, 1.5, 100, workspace=ws)
    prof = rfsf.rfsf_ts_profile_read(True)
    rfsf.rfsf_ts_profile_enable(False)
    assert prof["launches_rff_increments"] == projections
    assert prof["launches_sketch_fft_scan"] == (3 if projections else 4)
