"""The Gram's three-term bfloat16 products: every kernel and edge of its dispatch against 64-bit sums.

Bound of an entry: 32-bit summation in any order is within (K + 1) 2^-24 sum_k |a_k b_k|, and the three products of
terms that are left out are together within 2^-24 of each |a_k b_k| (mid*lo and lo*mid 2^-25 each at most, lo*lo next to
nothing): (K + 2) 2^-24 sum_k |a_k b_k|."""
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


@pytest.mark.parametrize("Nx,Ny,C,packed", [(40, 50, 100, False), (1000, 900, 600, True), (1100, 1030, 70, False),
                                            (2560, 2432, 1030, False), (2500, 2437, 40, True),
                                            (300, 0, 513, True), (1400, 0, 90, False), (3400, 0, 40, False), (3401, 0, 39, True)])
def test_nan_and_infinite_rows(Nx, Ny, C, packed):
    """What is NaN, infinite and finite in the 64-bit product is so in the 32-bit one, whichever column it comes from."""
    rng = np.random.default_rng(Nx + C)
    A = _operand(rng, Nx, C, packed).clamp(-1e4, 1e4)
    B = A if Ny == 0 else _operand(rng, Ny, C, packed).clamp(-1e4, 1e4)
    inf, nan = float("inf"), float("nan")
    for operand in (A, B):              # the column of the huge number: no product of it overflows but its square
        operand[:, 2] = operand[:, 2].clamp(-0.5, 0.5)
    for r, c in ((1, 0), (15, C - 1), (16, C // 2), (Nx // 2, 0), (Nx // 2 + 1, C - 1), (Nx - 1, 3)):
        A[r, c] = nan
    A[3, 1], A[5, C - 1], A[Nx // 3, 2], A[Nx - 2, C // 2] = inf, -inf, 3.4e38, inf
    A[8, 1:3] = torch.tensor([inf, -inf], device="cuda")
    A[20, :] = nan
    A[21, :] = inf
    if Ny:
        B[4, 0], B[Ny - 1, C - 1], B[Ny // 2, 7], B[11, 1] = nan, nan, nan, inf
        B[12, 1] = 0.0                  # against A's infinite rows: inf * 0
        B[Ny // 3, :] = nan
    want = A.double() @ B.double().T.contiguous()
    K = rfsf.rfsf_ts_gram(A) if Ny == 0 else rfsf.rfsf_ts_gram(A, B)
    assert torch.equal(torch.isnan(K), torch.isnan(want))
    assert torch.equal(torch.isposinf(K), torch.isposinf(want.float())) and torch.equal(torch.isneginf(K), torch.isneginf(want.float()))
    ok = torch.isfinite(want) & (want.abs() < 1e38)
    bound = (C + 2) * 2.0 ** -24 * (torch.nan_to_num(A, 0, 0, 0).double().abs() @ torch.nan_to_num(B, 0, 0, 0).double().abs().T.contiguous())
    assert bool((((K.double() - want).abs() <= bound) | ~ok).all())
    if Ny == 0:
        assert torch.equal(torch.nan_to_num(K, nan=1.25), torch.nan_to_num(K.T, nan=1.25))


@pytest.mark.parametrize("N,C", [(300, 513), (1000, 1025), (1400, 1025), (3000, 2049)])
def test_nan_takes_no_longer_than_numbers(N, C):
    """A sequence whose features are NaN, and a batch of nothing else: not much slower than numbers are (they were 15 to
    70 times slower when every such entry was summed up again). Best of five, and 50 us of slack for the smallest."""
    A = _operand(np.random.default_rng(N), N, C, False)

    def best(a, b):
        K = torch.empty((N, N), device="cuda")
        rfsf.rfsf_ts_gram(a, b, K=K)
        times = []
        for _ in range(5):
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            rfsf.rfsf_ts_gram(a, b, K=K)
            stop.record()
            stop.synchronize()
            times.append(start.elapsed_time(stop) * 1e3)
        return min(times)

    numbers = best(A, A)
    one, every = A.clone(), A.clone()
    one[N // 3, 1:] = float("nan")
    every[:, 1:] = float("nan")
    times = [best(one, one), best(A, one), best(every, every)]
    print(f"{N} x {C}: numbers {numbers:.1f} us, one row {times[0]:.1f}, of one operand {times[1]:.1f}, all {times[2]:.1f}")
    assert max(times) <= 2 * numbers + 50
