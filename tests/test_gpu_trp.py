"""RFSF-TRP on the GPU against the oracle, block-normalised error per level."""
import math

import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from paper_2501_07145_amd import binding
from tests.parity import FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


def _case(seed, N, L, d, M, F, Q, ls):
    rng = np.random.default_rng(seed)
    X = np.cumsum(rng.standard_normal((N, L, d)) / math.sqrt(L), axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    Z = rng.standard_normal((M, Q, 2 * F)).astype(np.float32)
    return X, W, Z, float(np.float32(ls))


def _run(X, W, Z, ls, **kw):
    out = rfsf.rfsf_trp_features(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), torch.from_numpy(Z).cuda(),
                                 ls, **kw)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("N,L,d,M,F,Q", [
    (16, 32, 3, 3, 32, 64),       # tiny-like
    (24, 100, 8, 4, 128, 256),    # small-like
    (5, 37, 5, 3, 24, 50),        # Q not a power of two, ragged everything
    (3, 9, 4, 2, 7, 33),          # odd F: 2F not a multiple of 4, plain GEMM path
    (2, 2, 3, 4, 16, 16),         # one increment
    (2, 1, 3, 2, 8, 8),           # no increments
    (1, 300, 2, 6, 16, 300),      # long, six levels, two component blocks
    (3, 30, 3, 1, 8, 12),         # one level; 29 increments in batches of eight
    (2, 23, 4, 5, 16, 1024),      # five levels, a whole 4 KB row of the projections per sequence
    (2, 18, 3, 7, 8, 36),         # seven levels: batches of three, sequences sharing a workgroup
    (2, 11, 3, 9, 8, 20),         # more than eight levels: the 16-level kernel, one step per batch
    (2, 14, 3, 12, 8, 18),        # the same with components that are no multiple of four
    (300, 5, 2, 2, 4, 8),         # many short sequences: 150 per workgroup
])
def test_trp_matches_oracle(oracle, N, L, d, M, F, Q):
    X, W, Z, ls = _case(N + L + Q, N, L, d, M, F, Q, ls=math.sqrt(d))
    got = _run(X, W, Z, ls).cpu().numpy()
    want = oracle.trp_features(X, W, Z, ls)
    err = block_errors(got, want, M, Q)
    print(f"N={N} L={L} d={d} M={M} F={F} Q={Q} block errors {err}")
    assert np.all(err <= FP32_BLOCK_TOL)


@pytest.mark.parametrize("F", [50, 7, 200, 65])
def test_products_of_all_levels_in_large_tiles(oracle, F):
    """So many rows that the levels' products take the 256 x 128 tiles, one level per grid row: rows on 16 bytes (2F = 100)
    and not (2F = 14), neither whole steps of 16 columns nor whole tiles of rows or of projections; from 128 columns on two
    terms instead of three (2F = 400, 130)."""
    N, L, M, Q = 2500, 8, 5, 200
    X, W, Z, ls = _case(F, N, L, 3, M, F, Q, math.sqrt(3))
    got = _run(X, W, Z, ls).cpu().numpy()
    sel = np.r_[0:40, 1020:1060, N - 40:N]
    err = block_errors(got[sel], oracle.trp_features(X[sel], W, Z, ls), M, Q)
    print(f"F={F}: block errors {err}")
    assert np.all(err <= FP32_BLOCK_TOL)
    assert np.all(got[:, 0] == 1.0) and np.all(np.isfinite(got))


@pytest.mark.parametrize("F", [200, 65])
def test_products_that_fall_back_to_three_terms(oracle, F):
    """Rows of Z that do not fit the scales of two terms, in some levels and tiles of the launch: from the outset (too small) and
    when the products are known (numbers far larger than those that are looked at)."""
    N, L, M, Q = 2500, 8, 5, 200
    X, W, Z, ls = _case(F, N, L, 3, M, F, Q, math.sqrt(3))
    Z[1, 150] *= np.float32(2.0 ** -95)
    Z[3, 5, 60::97] *= np.float32(2.0 ** 30)
    got = _run(X, W, Z, ls).cpu().numpy().astype(np.float64)
    sel = np.r_[0:40, 1020:1060, N - 40:N]
    got, want = got[sel], np.asarray(oracle.trp_features(X[sel], W, Z, ls), np.float64)
    for m in range(M):
        for part in ([150], [5], np.setdiff1d(np.arange(Q), [150, 5])):
            a, b = got[:, 1 + m * Q + np.array(part)], want[:, 1 + m * Q + np.array(part)]
            assert np.linalg.norm(a - b) <= FP32_BLOCK_TOL * np.linalg.norm(b), (m, part)


def test_trp_chunks_padding_and_errors(oracle):
    X, W, Z, ls = _case(3, 7, 12, 3, 2, 16, 20, 1.0)
    _, mn = rfsf.rfsf_trp_workspace_bytes(7, 12, 3, 2, 16, 20)
    rec2, _ = rfsf.rfsf_trp_workspace_bytes(2, 12, 3, 2, 16, 20)
    ws = torch.empty(mn + 2 * (rec2 - mn), dtype=torch.uint8, device="cuda")     # three sequences per chunk
    buf = torch.full((7, 41 + 3), -5.0, dtype=torch.float32, device="cuda")
    _run(X, W, Z, ls, out=buf, workspace=ws)
    assert torch.all(buf[:, 41:] == -5.0)
    assert np.all(block_errors(buf[:, :41].cpu().numpy(), oracle.trp_features(X, W, Z, ls), 2, 20) <= FP32_BLOCK_TOL)
    with pytest.raises(binding.RfsfTsError) as e:
        _run(X, W, Z, ls, workspace=torch.empty(mn - 1, dtype=torch.uint8, device="cuda"))
    assert e.value.code == -6


def test_trp_more_sequences_than_one_launch_may_take(oracle):
    # 70000 sequences: a launch takes at most 65535, so the call must split the batch even though the workspace
    # would hold it whole
    N, L, d, M, F, Q = 70000, 3, 2, 2, 2, 4
    X, W, Z, ls = _case(11, N, L, d, M, F, Q, 1.0)
    got = _run(X, W, Z, ls).cpu().numpy()
    sel = np.r_[0:40, 34990:35010, 65530:65540, N - 40:N]
    want = oracle.trp_features(X[sel], W, Z, ls)
    assert np.all(block_errors(got[sel], want, M, Q) <= FP32_BLOCK_TOL)
    assert np.all(got[:, 0] == 1.0) and np.all(np.isfinite(got))


@pytest.mark.parametrize("L,M,F,Q", [
    (4001, 1, 16, 33), (10001, 1, 32, 33), (20001, 1, 64, 40),       # the three small-tile product kernels
    (20001, 5, 16, 200), (20001, 5, 7, 200),                         # large tiles, rows on 16 bytes and not
    (20001, 5, 64, 200), (20001, 5, 65, 200),                        # two terms
])
def test_errors_of_the_products_do_not_add_up_over_time(L, M, F, Q):
    """Level 1 is the sum of all projected increments, Z (phi(x_T) - phi(x_0)): on noise no larger than one of its T
    summands, so that a rounding error of the products with a sign of its own would grow past those that cancel. Bound:
    T independent errors of a 32-bit sum of products, 2^-24 of its root mean square each, times four."""
    rng = np.random.default_rng(L + F)
    X = rng.standard_normal((1, L, 1)).astype(np.float32)
    W = rng.standard_normal((M, 1, F)).astype(np.float32)
    Z = rng.standard_normal((M, Q, 2 * F)).astype(np.float32)
    got = _run(X, W, Z, 1.0).cpu().numpy()[0, 1:1 + Q].astype(np.float64) * math.sqrt(Q)

    theta = X[0].astype(np.float64) @ W[0].astype(np.float64)
    phi = np.concatenate([np.cos(theta), np.sin(theta)], axis=1) / math.sqrt(F)
    z = Z[0].astype(np.float64).T
    size = math.sqrt((((phi[1:2000] - phi[:1999]) @ z) ** 2).mean())
    err = math.sqrt(((got - (phi[-1] - phi[0]) @ z) ** 2).mean()) / (math.sqrt(L - 1) * size)
    print(f"L={L} M={M} F={F} Q={Q}: {err * 2 ** 24:.2f} units")
    assert err <= 4 * 2.0 ** -24


@pytest.mark.parametrize("N,L,Q", [(6, 40, 33), (300, 2, 8), (1, 300, 20)])
def test_nothing_is_computed_from_what_the_workspace_held(N, L, Q):
    """A batch has one increment less than points. What the workspace held in the last row enters no product:
    infinite, it would leave NaN behind in the workspace (with mixed signs in Z), and NaN takes time."""
    M, F = 3, 12
    X, W, Z, ls = _case(N + L, N, L, 3, M, F, Q, 1.0)
    ws = torch.zeros(rfsf.rfsf_trp_workspace_bytes(N, L, 3, M, F, Q)[0] // 4 * 4, dtype=torch.uint8, device="cuda")
    want = _run(X, W, Z, ls, workspace=ws).clone()
    ws.view(torch.float32).fill_(float("inf"))
    got = _run(X, W, Z, ls, workspace=ws)
    assert torch.equal(got, want)
    assert not bool(torch.isnan(ws.view(torch.float32)).any())


def test_the_cut_in_time_does_not_depend_on_the_workspace():
    """Sequences are cut by the shape of the batch, not by how many of them a launch takes: the same bits for a batch as a
    whole and for one sequence at a time. (So many components that both run the same product kernel, and the first
    sequence, whose rows are the first ones of their product either way.)"""
    N, L, M, F, Q = 2, 129, 2, 16, 32768
    X, W, Z, ls = _case(5, N, L, 3, M, F, Q, 1.0)
    rec, mn = rfsf.rfsf_trp_workspace_bytes(N, L, 3, M, F, Q)
    assert mn < rec
    runs = [_run(X, W, Z, ls, workspace=torch.empty(n, dtype=torch.uint8, device="cuda")) for n in (rec, mn)]
    assert torch.equal(runs[0][0], runs[1][0])
