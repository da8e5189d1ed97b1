"""The Gram's two-term 16-bit products (large tiles, 128 columns and more): edges, scales and what does not fit them.

Bound of an entry: 32-bit summation is within (K + 1) 2^-24 sum_k |a_k b_k|; a number's two terms are within 2^-22 of it or
within 2^-33 of its row's largest number, for both operands, and the product that is left out is within 2^-22 of each
|a_k b_k|: (K + 13) 2^-24 sum_k |a_k b_k| + 2^-33 (max|a| sum_k |b_k| + max|b| sum_k |a_k|)."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

pytestmark = pytest.mark.gpu


def _operand(rng, rows, cols, packed, kind):
    ld = cols if packed else (cols + 3) // 4 * 4
    a = rng.standard_normal((rows, ld)).astype(np.float32)
    if kind == "wide":
        a *= np.exp2(rng.integers(-12, 12, (rows, ld)))
    elif kind == "rising":              # every column larger than the one before
        a *= np.exp2(np.arange(ld) * (24.0 / ld))
    elif kind == "hidden":              # numbers that no sample sees, far beyond the scale
        a[:, 60::97] *= 2.0 ** 30
    elif kind == "zeros":               # rows that are zero wherever they are sampled, rows that are zero
        a[::3, :] = 0.0
        a[::6, 52:60] = 1.5
    elif kind == "small":
        a *= 2.0 ** -60
        a[1::2] *= 2.0 ** -50           # beyond the scales' range
    elif kind == "large":
        a[::2] *= 2.0 ** 50
    return torch.from_numpy(a.astype(np.float32)).cuda()[:, :cols]


def _check(K, A, B):
    a, b = A.double(), B.double()
    n = a.shape[1]
    bound = (n + 13) * 2.0 ** -24 * (a.abs() @ b.abs().T.contiguous())
    bound += 2.0 ** -33 * (a.abs().amax(1)[:, None] * b.abs().sum(1)[None] + a.abs().sum(1)[:, None] * b.abs().amax(1)[None])
    bound += 2.0 ** -149
    err = (K.double() - a @ b.T.contiguous()).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("Nx,Ny,C,packed", [(2600, 2700, 128, False), (2561, 2689, 129, True), (2600, 2690, 143, False),
                                            (2816, 2560, 144, True), (2600, 2561, 175, False), (2600, 2600, 1030, True)])
@pytest.mark.parametrize("kind", ["normal", "wide", "rising", "hidden", "zeros", "small", "large"])
def test_two_operands(Nx, Ny, C, packed, kind):
    rng = np.random.default_rng(Nx + Ny + C)
    A, B = _operand(rng, Nx, C, packed, kind), _operand(rng, Ny, C, packed, "normal" if kind == "small" else kind)
    K = torch.full((Nx, Ny + 3), -3.0, device="cuda")
    _check(rfsf.rfsf_ts_gram(A, B, K=K[:, :Ny]), A, B)
    assert bool((K[:, Ny:] == -3.0).all())


@pytest.mark.parametrize("N,C,packed", [(3585, 257, True), (3700, 400, False), (3841, 144, False)])
@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("kind", ["wide", "hidden"])
def test_one_operand_is_symmetric(N, C, packed, pad, kind):
    A = _operand(np.random.default_rng(N), N, C, packed, kind)
    K = torch.full((N, N + pad), -3.0, device="cuda")
    rfsf.rfsf_ts_gram(A, K=K[:, :N])
    _check(K[:, :N], A, A)
    assert torch.equal(K[:, :N], K[:, :N].T)
    assert bool((K[:, N:] == -3.0).all())


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("up_a,up_b", [(-62, -62), (-66, -66), (-80, -50), (-70, 70), (80, -75), (40, 60)])
def test_scales_of_both_rows_together(up_a, up_b, packed):
    """Rows whose scales multiply to more or less than a float holds, while the products of the rows do not."""
    rng = np.random.default_rng(1000 + up_a)
    A, B = _operand(rng, 2600, 1030, packed, "normal"), _operand(rng, 2700, 1030, packed, "normal")
    A *= 2.0 ** up_a
    B *= 2.0 ** up_b
    _check(rfsf.rfsf_ts_gram(A, B), A, B)


@pytest.mark.parametrize("both", [0.0, 2.0 ** -11])
@pytest.mark.parametrize("up_a,up_b", [(73, 73), (80, 80), (95, 60)])
def test_large_rows_that_hardly_meet(up_a, up_b, both):
    """A has even columns and B odd ones, and both one that they share: sums of two or three ordinary numbers, or zero."""
    rng = np.random.default_rng(up_a)
    A, B = _operand(rng, 2600, 300, False, "normal"), _operand(rng, 2700, 300, False, "normal")
    A[:, 1::2] = 0.0
    B[:, ::2] = 0.0
    if up_a + up_b < 150:
        A[:, 101], B[:, 101] = both, -both
    A *= 2.0 ** up_a
    B *= 2.0 ** up_b
    K = rfsf.rfsf_ts_gram(A, B)
    want = (A.double() @ B.double().T.contiguous()).float()
    if both == 0.0 or up_a + up_b >= 150:
        assert bool((K == 0.0).all())
    else:
        assert torch.equal(K, want)                          # one product of powers of two per entry


def _check_products(K, A, B):
    """Against the products of the entry alone: (K + 13) 2^-24 of them as above, and K / 32 (the sampled products) more."""
    a, b = A.double(), B.double()
    bound = (1.04 * a.shape[1] + 13) * 2.0 ** -24 * (a.abs() @ b.abs().T.contiguous()) + 2.0 ** -149
    err = (K.double() - a @ b.T.contiguous()).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("kind", ["one", "one_hidden", "half", "one_row", "few_rows"])
@pytest.mark.parametrize("C,packed", [(128, False), (300, True), (1030, False)])
def test_large_numbers_against_zeros(C, packed, kind, swap):
    """Rows with a range wider than two terms hold, whose large numbers meet zeros: what is left is made of their small ones."""
    rng = np.random.default_rng(C)
    A, B = _operand(rng, 2600, C, packed, "normal"), _operand(rng, 2700, C, packed, "normal")
    where = {"one": 3, "one_hidden": 50}.get(kind, 20)
    if kind == "half":
        A[:, C // 2:] *= 2.0 ** -20
        B[:, :C // 2] = 0.0
    else:
        small = {"one_row": slice(1500, 1501), "few_rows": slice(7, 2600, 301)}.get(kind, slice(None))
        A[small] *= 2.0 ** -20
        A[small, where] = 1.0
        B[:, where] = 0.0
    K = rfsf.rfsf_ts_gram(B, A).T if swap else rfsf.rfsf_ts_gram(A, B)
    _check_products(K, A, B)


@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("up", [-112, -60])
def test_rows_that_are_zero_where_they_are_sampled(up, swap):
    """Small numbers in such rows enter with all their bits, as they do in others."""
    rng = np.random.default_rng(-up)
    A, B = _operand(rng, 2600, 300, True, "normal"), _operand(rng, 2700, 300, False, "normal")
    A[5::7] = 0.0
    A[5::35, 52:60] = torch.from_numpy(rng.uniform(1.0, 2.0, (75, 8)).astype(np.float32) * np.float32(2.0 ** up)).cuda()
    K = rfsf.rfsf_ts_gram(B, A).T if swap else rfsf.rfsf_ts_gram(A, B)
    _check_products(K, A, B)
    assert bool((K[12::35] == 0.0).all())


def test_unit_vectors_give_the_numbers_themselves():
    A = _operand(np.random.default_rng(3), 2600, 300, False, "wide")
    K = rfsf.rfsf_ts_gram(A, torch.eye(300, device="cuda").repeat(9, 1))
    assert torch.equal(K, A.repeat(1, 9))


def test_error_is_no_larger_than_three_terms():
    """2-norm of the error over that of the result; three terms had 1.63e-7, 3.0e-7 and 5.3e-7 here (the rows of the first
    two are normal numbers, the last has a column of ones), a margin of a tenth for other seeds."""
    for n, C, limit in ((3000, 128, 1.8e-7), (3000, 400, 3.3e-7), (4000, 1001, 5.8e-7)):
        A = _operand(np.random.default_rng(C), n, C, False, "normal")
        if C == 1001:
            A = A / C ** 0.5
            A[:, 0] = 1.0
        want = A.double() @ A.double().T.contiguous()
        err = rfsf.rfsf_ts_gram(A, A.clone()).double() - want
        assert float(err.norm() / want.norm()) <= limit, (C, float(err.norm() / want.norm()))


@pytest.mark.parametrize("n", [2500, 3000, 4000])
def test_sums_are_not_joined_for_speed(n):
    """Sizes at which small tiles, which add up in several sums, and one sum of two terms take turns: the error of small tiles
    (5.0e-7 here, measured, and 9.4e-7 in large ones; the limit lies between)."""
    A = _operand(np.random.default_rng(n), n, 5121, False, "normal") / 5121 ** 0.5
    A[:, 0] = 1.0
    want = A.double() @ A.double().T.contiguous()
    err = rfsf.rfsf_ts_gram(A).double() - want
    assert float(err.norm() / want.norm()) <= 7e-7, float(err.norm() / want.norm())


def test_nan_and_infinite_rows():
    rng = np.random.default_rng(5)
    A, B = _operand(rng, 2600, 500, False, "normal"), _operand(rng, 2700, 500, False, "normal")
    inf, nan = float("inf"), float("nan")
    for r, c in ((1, 0), (300, 499), (700, 250), (2599, 3)):
        A[r, c] = nan
    A[900, 1], A[1300, 499], A[1301, 77], A[2000, 60] = inf, -inf, 3.4e38, inf
    B[40, 200], B[2699, 499], B[1000, 9] = nan, nan, inf
    B[12, 1] = 0.0                      # against A's infinite row: inf * 0
    want = A.double() @ B.double().T.contiguous()
    K = rfsf.rfsf_ts_gram(A, B)
    assert torch.equal(torch.isnan(K), torch.isnan(want))
    ok = torch.isfinite(want) & (want.abs() < 1e38)
    assert torch.equal(torch.isposinf(K) & ~ok, torch.isposinf(want.float()) & ~ok)
    assert torch.equal(torch.isneginf(K) & ~ok, torch.isneginf(want.float()) & ~ok)
    bound = (500 + 13) * 2.0 ** -24 * (torch.nan_to_num(A, 0, 0, 0).double().abs() @ torch.nan_to_num(B, 0, 0, 0).double().abs().T.contiguous())
    assert bool((((K.double() - want).abs() <= bound + 1e-6) | ~ok).all())
