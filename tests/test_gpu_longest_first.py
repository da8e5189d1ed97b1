"""Batches of sequences with lengths of their own are taken by length, the longest first: each workgroup finds its sequence by counting.
Every sequence is still computed exactly once, with the same sums; the sizes sit at the edges of the rule: the smallest batch it
applies to and the one below, the least work and a pair of steps less, the largest batch that fits the registers of three and four
wavefronts and the next, equal lengths, lengths out of range, and a class with all sequences but one. Small sequences and pieces are taken in
order of their numbers, which gives the same rows."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

pytestmark = pytest.mark.gpu


def _lengths(kind, N, L, rng):
    if kind == "any":
        return rng.integers(1, L + 1, size=N)
    if kind == "half":
        return rng.integers((L + 1) // 2, L + 1, size=N)
    if kind == "outside":
        return rng.integers(-3, L + 4, size=N)
    lengths = np.full(N, L)
    if kind == "one short":
        lengths[N // 2] = 1
    if kind == "one long":
        lengths[:] = 2
        lengths[N - 1] = L
    return lengths


@pytest.mark.parametrize("N,L,d,M,F,D,order,kind", [
    shape + (kind,) for kind in ("any", "equal") for shape in [
        (256, 300, 3, 5, 60, 512, 1), (257, 300, 3, 5, 60, 512, 1), (1100, 60, 3, 3, 60, 1024, 1), (520, 66, 3, 4, 100, 500, 2),
        (64, 2100, 3, 3, 60, 512, 1), (200, 900, 3, 4, 40, 500, 1), (1200, 250, 3, 5, 60, 64, 2),          # pieces; grouped transforms
        (300, 108, 3, 2, 20, 512, 1), (300, 110, 3, 2, 20, 512, 1), (260, 62, 3, 2, 30, 1000, 3),
        (1536, 48, 3, 3, 20, 512, 1), (1537, 48, 3, 3, 20, 512, 1),          # the most sequences for their work, and one more
        (400, 120, 2, 5, 18, 64, 1), (300, 301, 2, 5, 50, 100, 1)]           # single wavefronts, two and three pieces that start with any of them
] + [shape + (kind,) for kind in ("any", "half", "equal", "outside", "one short", "one long") for shape in [
    (256, 40, 3, 5, 120, 512, 1), (257, 40, 3, 5, 120, 512, 1), (300, 333, 3, 4, 250, 500, 2), (90, 300, 5, 5, 50, 100, 1),
    (320, 10, 3, 3, 60, 1024, 1), (321, 10, 3, 3, 60, 1024, 1), (300, 35, 9, 2, 100, 1024, 3), (270, 24, 3, 3, 40, 2048, 1),
    (6144, 192, 2, 3, 8, 512, 1), (6145, 193, 2, 3, 8, 512, 1), (8192, 256, 2, 4, 8, 500, 1), (8193, 257, 2, 4, 8, 500, 1),
    (700, 33, 12, 3, 60, 64, 2), (2048, 80, 2, 1, 40, 512, 1),
]])
def test_every_sequence_once(N, L, d, M, F, D, order, kind):
    """Rows do not depend on the place of their sequence in the batch, and are those of whole sequences whose last point stays."""
    rng = np.random.default_rng(N + L + D)
    X = torch.from_numpy(np.cumsum(rng.standard_normal((N, L, d)) * 0.2, axis=1).astype(np.float32)).cuda()
    W = torch.from_numpy(rng.standard_normal((M, d, F)).astype(np.float32)).cuda()
    hash_ = torch.from_numpy(rng.integers(0, D, size=(M, 2 * F)).astype(np.int32)).cuda()
    sign = torch.from_numpy((2.0 * rng.integers(0, 2, size=(M, 2 * F)) - 1.0).astype(np.float32)).cuda()
    lengths = torch.from_numpy(_lengths(kind, N, L, rng).astype(np.int64))
    got = rfsf.rfsf_ts_features(X, W, hash_, sign, 1.5, D, order=order, lengths=lengths.cuda())
    # the same batch in another order of its sequences: every row is the same to the bit
    turned = torch.from_numpy(rng.permutation(N))
    again = rfsf.rfsf_ts_features(X[turned.cuda()].contiguous(), W, hash_, sign, 1.5, D, order=order, lengths=lengths[turned].cuda())
    assert torch.equal(again, got[turned.cuda()])
    # and as whole sequences whose last point is repeated: the added increments are zero
    stay = lengths.clamp(1, L) - 1
    t = torch.minimum(torch.arange(L)[None, :], stay[:, None]).cuda()
    whole = rfsf.rfsf_ts_features(torch.gather(X, 1, t[:, :, None].expand(N, L, d)).contiguous(), W, hash_, sign, 1.5, D, order=order)
    scale = whole.double().square().mean(0).sqrt().max()
    # (sums in another order where wavefronts or pieces share a sequence out: 1e-5 of the largest column, as against the oracle)
    assert float((got - whole).abs().max()) <= 1e-5 * max(1.0, float(scale))
