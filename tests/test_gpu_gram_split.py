"""The Gram's three-term bfloat16 products: every kernel and edge of its dispatch against 64-bit sums.

Bound of an entry: 32-bit summation in any order is within (K + 1) 2^-24 sum_k |a_k b_k|, and the three products of
terms that are left out are within 2^-25 of each |a_k b_k|: (K + 2) 2^-24 sum_k |a_k b_k|."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf

pytestmark = pytest.mark.gpu


def _operand(rng, rows, cols, packed, offset=0):
    ld = cols if packed else (cols + 3) // 4 * 4
    a = (rng.standard_normal((rows, ld)) * np.exp2(rng.integers(-12, 12, (rows, ld)))).astype(np.float32)
    flat = torch.zeros(rows * ld + offset, dtype=torch.float32, device="cuda")
    flat[offset:] = torch.from_numpy(a.reshape(-1)).cuda()
    return flat[offset:].view(rows, ld)[:, :cols]


def _check(K, A, B):
    a, b = A.double(), B.double()
    bound = (a.shape[1] + 2) * 2.0 ** -24 * (a.abs() @ b.abs().T)
    err = (K.double() - a @ b.T).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("Nx,Ny,C,packed", [
    (1, 1, 1, True), (1, 33, 31, True), (32, 31, 32, False), (33, 65, 33, True),        # 32 x 32 tiles, steps of 32
    (5, 70, 255, False), (64, 64, 256, True), (40, 40, 289, False),                     # eight wavefronts share K
    (1025, 1030, 63, True), (1100, 1027, 64, False), (1089, 1089, 130, True),           # 64 x 64 tiles
    (2560, 2432, 15, False), (2561, 2433, 16, True), (2500, 2560, 17, True),            # 256 x 128 tiles, steps of 16
    (2500, 2561, 31, False), (2304, 2688, 48, False), (2500, 2560, 50, True), (2500, 2560, 66, False),
])
def test_two_operands(Nx, Ny, C, packed):
    rng = np.random.default_rng(Nx + Ny + C)
    A, B = _operand(rng, Nx, C, packed), _operand(rng, Ny, C, packed, offset=1 if packed else 0)
    _check(rfsf.rfsf_ts_gram(A, B), A, B)


@pytest.mark.parametrize("N,C,packed", [(31, 40, True), (65, 100, False), (1441, 33, True), (1500, 70, False),
                                        (3400, 49, False), (3585, 17, True), (5121, 40, True), (5000, 64, False)])
@pytest.mark.parametrize("pad", [0, 3])
def test_one_operand_is_symmetric(N, C, packed, pad):
    A = _operand(np.random.default_rng(N), N, C, packed)
    K = torch.full((N, N + pad), -3.0, device="cuda")
    rfsf.rfsf_ts_gram(A, K=K[:, :N])
    _check(K[:, :N], A, A)
    assert torch.equal(K[:, :N], K[:, :N].T)
    assert bool((K[:, N:] == -3.0).all())


@pytest.mark.parametrize("N", [40, 1100, 3400])
def test_infinite_and_huge_operands(N):
    """Numbers whose split is not finite: an infinite one, and one above the largest bfloat16 number."""
    A = _operand(np.random.default_rng(N), N, 40, False)
    B = torch.ones_like(A)
    B[:, 1:] = 0.0
    A[3, 0], A[7, 0], A[9, 0] = float("inf"), float("-inf"), 3.4e38
    A[11, 20] = float("nan")
    want = A.double() @ B.double().T
    K = rfsf.rfsf_ts_gram(A, B)
    for r in (3, 7, 9, 11):            # inf * 0 is NaN in the sum of every column of B but those that are not zero
        assert torch.equal(torch.nan_to_num(K[r], nan=1.25), torch.nan_to_num(want[r].float(), nan=1.25)), r
    B[:, 1:] = 0.5
    want, K = A.double() @ B.double().T, rfsf.rfsf_ts_gram(A, B)
    assert torch.equal(torch.isinf(K[[3, 7]]), torch.isinf(want[[3, 7]].float())) and bool(torch.isnan(K[11]).all())
    assert bool(torch.isfinite(K[9]).all())
