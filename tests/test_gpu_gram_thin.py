"""Gram of a few rows with others, and of few tiles of 16 x 16: both sides of every rule, columns around whole steps, packed rows, and
what is not finite."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

pytestmark = pytest.mark.gpu


def _gram(A, B):
    K = torch.full((A.shape[0], B.shape[0] + 3), -7.0, device="cuda")
    rfsf.rfsf_ts_gram(A, B, K=K[:, :B.shape[0]])
    assert bool((K[:, B.shape[0]:] == -7.0).all())
    return K[:, :B.shape[0]]


@pytest.mark.parametrize("few,many,cols", [
    (1, 1, 320), (1, 2, 319), (1, 1000, 1025), (2, 7, 511), (3, 100, 512), (4, 2047, 513), (4, 2048, 321), (5, 2047, 767), (8, 33, 1024),
    (8, 2048, 2047), (8, 2048, 2048), (6, 8191, 2049), (5, 8192, 2050), (8, 8195, 2051), (9, 50, 1025), (1, 9000, 400), (8, 8, 5121),
])
def test_sums_match_64_bits(few, many, cols):
    """A sum of products of `cols` numbers in 32 bits: a few times 2^-24 of the root sum of their squares, sqrt(cols) of them at random
    signs; 2e-6 is the tolerance of the larger tiles' tests too."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(few * many + cols)
    A = torch.randn((few, cols), generator=gen, device="cuda")
    B = torch.randn((many, cols), generator=gen, device="cuda")
    want = A.double() @ B.double().T
    scale = (A.double() ** 2).sum(1).sqrt()[:, None] * (B.double() ** 2).sum(1).sqrt()[None, :]
    wide = torch.zeros((many, cols + 5), device="cuda")[:, 1:cols + 1]           # a stride and an alignment of its own
    wide.copy_(B)
    for a, b, w, s in ((A, B, want, scale), (B, A, want.T, scale.T), (A, wide, want, scale)):
        got = _gram(a, b)
        assert float(((got.double() - w) / s).abs().max()) <= 2e-6
        assert torch.equal(got, _gram(a, b))
    own = _gram(A, A)
    assert torch.equal(own, own.T)


@pytest.mark.parametrize("few,many,cols,thin", [
    (8, 2047, 867, False), (8, 2047, 868, True), (5, 60, 583, False), (5, 60, 584, True), (8, 4096, 2048, True), (8, 4097, 2049, False),
    (6, 6144, 2048, True), (6, 6145, 2049, False), (5, 8192, 5121, False), (8, 8193, 2048, True), (8, 12289, 2303, False), (5, 14000, 2304, True),
    (4, 8192, 8192, True), (4, 8192, 8193, False), (3, 6144, 11000, True), (4, 8193, 8200, True), (2, 7000, 9700, True),
])
def test_tiles_are_taken_where_they_are_faster(few, many, cols, thin):
    """A ninth row leaves the others in tiles, whose rows do not depend on each other: the same bits only where both are."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(many + cols)
    A = torch.randn((9, cols), generator=gen, device="cuda")
    B = torch.randn((many, cols), generator=gen, device="cuda")
    for got, tiles in ((_gram(A[:few], B), _gram(A, B)[:few]), (_gram(B, A[:few]), _gram(B, A)[:, :few])):
        assert torch.equal(got, tiles) != thin
        assert float((got - tiles).abs().max()) <= 2e-6 * 2 * cols


def test_what_is_not_finite_stays_in_its_entries():
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    A, B = torch.rand((3, 700), generator=gen, device="cuda"), torch.rand((40, 700), generator=gen, device="cuda")
    want = _gram(A, B)
    B[5, 699], B[7, 3] = float("nan"), float("inf")
    got = _gram(A, B)
    assert bool(torch.isnan(got[:, 5]).all()) and bool(torch.isinf(got[:, 7]).all())
    keep = [j for j in range(40) if j not in (5, 7)]
    assert torch.equal(got[:, keep], want[:, keep])


@pytest.mark.parametrize("Nx,Ny,cols", [
    (9, 9, 65), (16, 16, 193), (17, 15, 31), (31, 33, 1025), (100, 100, 257), (256, 256, 129), (256, 257, 129), (40, 1300, 511), (9, 4096, 300),
    (352, 0, 97), (353, 0, 97), (20, 0, 2049),
])
def test_few_tiles(Nx, Ny, cols):
    """The bound of the larger tiles' sums: a random walk of 1 + K / 32 roundings of 2^-24 of r = sqrt(sum a^2 b^2) + |sum a b|, eight times."""
    rng = np.random.default_rng(Nx + cols)
    A = rng.standard_normal((Nx, cols)).astype(np.float32)
    B = A if Ny == 0 else rng.standard_normal((Ny, cols)).astype(np.float32)
    a = torch.from_numpy(A).cuda()
    got = (rfsf.rfsf_ts_gram(a) if Ny == 0 else rfsf.rfsf_ts_gram(a, torch.from_numpy(B).cuda())).cpu().numpy()
    A, B = A.astype(np.float64), B.astype(np.float64)
    r = np.sqrt((A ** 2) @ (B ** 2).T) + np.abs(A @ B.T)
    assert (np.abs(got - A @ B.T) / (8 * np.sqrt(1 + cols / 32) * 2.0 ** -24 * r)).max() <= 1
    if Ny == 0:
        assert np.array_equal(got, got.T)


def test_few_tiles_with_what_is_not_finite():
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    A, B = torch.rand((20, 333), generator=gen, device="cuda"), torch.rand((50, 333), generator=gen, device="cuda")
    want = rfsf.rfsf_ts_gram(A, B).clone()
    B[5, 332], B[7, 3] = float("nan"), float("inf")
    got = rfsf.rfsf_ts_gram(A, B)
    assert bool(torch.isnan(got[:, 5]).all()) and bool(torch.isinf(got[:, 7]).all())
    keep = [j for j in range(50) if j not in (5, 7)]
    assert torch.equal(got[:, keep], want[:, keep])
