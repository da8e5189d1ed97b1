"""RFSF-TRP keeps one row per increment: rows of increments close up behind a sequence's last point. Sequences of every length around
the 32 rows of a tile and the 31, 63, 127 and 255 increments of a workgroup's range, in all three projection kernels."""
import math

import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from tests.parity import FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [2, 3, 5, 31, 32, 33, 34, 64, 65, 255, 256, 257])
@pytest.mark.parametrize("d,bf16", [(3, False), (66, False), (3, True)])
def test_rows_close_up_behind_every_sequence(oracle, L, d, bf16):
    """Ranges of 255 increments on the vector units (66 channels), of 31, a tile, on the matrix units, where these batches are small."""
    N, M, F, Q = 2 + 600 // L, 3, 20, 24
    rng = np.random.default_rng(L)
    X = np.cumsum(rng.standard_normal((N, L, d)) / math.sqrt(L), axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    if bf16:                                                 # operands that the rounding leaves as they are
        X = (np.round(X * 64) / 64).astype(np.float32)
        W = (np.round(W * 16) / 16).astype(np.float32)
    Z = rng.standard_normal((M, Q, 2 * F)).astype(np.float32)
    ls = float(np.float32(2.0 if bf16 else math.sqrt(d)))
    got = rfsf.rfsf_trp_features(*(torch.from_numpy(a).cuda() for a in (X, W, Z)), ls, rff_bf16=bf16).cpu().numpy()
    want = oracle.trp_features(X, W, Z, ls)
    assert np.all(block_errors(got, want, M, Q) <= FP32_BLOCK_TOL)


@pytest.mark.parametrize("L", [2, 3, 5, 31, 32, 33, 34, 62, 63, 64, 65, 254, 255, 256, 257])
@pytest.mark.parametrize("rows", [2 * 255, 5 * 255, 9 * 255, 33 * 255])
@pytest.mark.parametrize("bf16", [False, True])
def test_ranges_of_several_tiles_on_the_matrix_units(oracle, L, rows, bf16):
    """63 slabs of 128 frequencies: 2 ranges of 255 increments (126 to 189 workgroups) are taken 63 at a time, two tiles, 5 (315, 378) 127, 9 (567,
    630) 63 again and 33 (2079 and more) as they are, eight tiles.
    A row out of its place would move those of all later sequences; some are compared, in the middle and at the end."""
    M, d, F, Q = 4, 3, 2000, 8
    N = rows // L + 1
    rng = np.random.default_rng(L + rows)
    X = np.cumsum(rng.standard_normal((N, L, d)) / math.sqrt(L), axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    if bf16:                                                 # operands that the rounding leaves as they are
        X = (np.round(X * 64) / 64).astype(np.float32)
        W = (np.round(W * 16) / 16).astype(np.float32)
    Z = rng.standard_normal((M, Q, 2 * F)).astype(np.float32)
    got = rfsf.rfsf_trp_features(*(torch.from_numpy(a).cuda() for a in (X, W, Z)), 2.0, rff_bf16=bf16).cpu().numpy()
    assert np.all(np.isfinite(got))
    few = max(2, 200 // L)
    sel = np.unique(np.clip(np.r_[0:few, N // 3:N // 3 + few, N // 2:N // 2 + few, N - few:N], 0, N - 1))
    want = oracle.trp_features(X[sel], W, Z, 2.0)
    assert np.all(block_errors(got[sel], want, M, Q) <= FP32_BLOCK_TOL)


@pytest.mark.parametrize("N,L,Q", [(16, 3, 200), (40, 2, 200), (300, 2, 200), (400, 2, 200), (700, 2, 200), (2400, 2, 200), (2400, 3, 200), (3000, 2, 72)])
def test_short_sequences_on_both_sides_of_the_kinds_of_tiles(oracle, N, L, Q):
    """The products' tiles are chosen by the increments, half as many as points here."""
    M, F = 5, 64
    rng = np.random.default_rng(N)
    X = rng.standard_normal((N, L, 3)).astype(np.float32)
    W = rng.standard_normal((M, 3, F)).astype(np.float32)
    Z = rng.standard_normal((M, Q, 2 * F)).astype(np.float32)
    got = rfsf.rfsf_trp_features(*(torch.from_numpy(a).cuda() for a in (X, W, Z)), 1.7).cpu().numpy()
    want = oracle.trp_features(X, W, Z, 1.7)
    levels = min(M, L - 1)                                   # (no more steps than levels: blocks of zeros)
    assert np.all(block_errors(got, want, M, Q)[:levels] <= FP32_BLOCK_TOL)
    assert not np.any(got[:, 1 + levels * Q:])


@pytest.mark.parametrize("L", [64, 65])
@pytest.mark.parametrize("d,bf16", [(8, False), (9, False), (40, False), (66, False), (16, True), (100, True)])
def test_rows_are_kept_from_65_points_and_9_channels_on(oracle, L, d, bf16):
    """Whole sequences, and 3 of 200 and more points in pieces, whose sums take the place of their rows."""
    M, F, Q = 5, 30, 36
    rng = np.random.default_rng(L + d)
    for N, points in ((150, L), (3, 3 * L + 8)):
        X = np.cumsum(rng.standard_normal((N, points, d)) / math.sqrt(points), axis=1).astype(np.float32)
        W = rng.standard_normal((M, d, F)).astype(np.float32)
        if bf16:
            X = (np.round(X * 64) / 64).astype(np.float32)
            W = (np.round(W * 16) / 16).astype(np.float32)
        Z = rng.standard_normal((M, Q, 2 * F)).astype(np.float32)
        got = rfsf.rfsf_trp_features(*(torch.from_numpy(a).cuda() for a in (X, W, Z)), math.sqrt(d), rff_bf16=bf16).cpu().numpy()
        want = oracle.trp_features(X, W, Z, math.sqrt(d))
        assert np.all(block_errors(got, want, M, Q) <= FP32_BLOCK_TOL)


@pytest.mark.parametrize("N,L,d", [(6, 70, 9), (1, 300, 20), (40, 64, 9), (5, 66, 70)])
def test_rows_that_are_kept_hold_nothing_of_the_workspace(N, L, d):
    """Steps from one sequence into the next are computed from the points where rows are kept; the batch's last row is in no product."""
    M, F, Q = 3, 12, 20
    rng = np.random.default_rng(N + L)
    X, W, Z = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda() for s in ((N, L, d), (M, d, F), (M, Q, 2 * F)))
    ws = torch.zeros(rfsf.rfsf_trp_workspace_bytes(N, L, d, M, F, Q)[0] // 4 * 4, dtype=torch.uint8, device="cuda")
    want = rfsf.rfsf_trp_features(X, W, Z, math.sqrt(d), workspace=ws).clone()
    ws.view(torch.float32).fill_(float("inf"))
    got = rfsf.rfsf_trp_features(X, W, Z, math.sqrt(d), workspace=ws)
    assert torch.equal(got, want)
    assert not bool(torch.isnan(ws.view(torch.float32)).any())
