"""Sketch tables: the coordinates of a level sorted into buckets, built by workgroups of the projection launch or, where
that launch cannot take them, by one of their own. Level 1 and 2 blocks against the oracle where the sorting can go
wrong: fewer and more buckets than coordinates, numbers of coordinates around the workgroup's size, all in one bucket."""
import numpy as np
import pytest
import torch

import paper_2501_07145_amd as rfsf
from tests.parity import FP32_BLOCK_TOL, block_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,F,D,kind", [
    (3, 1, 64, "random"),
    (3, 127, 64, "random"), (3, 128, 64, "random"), (3, 129, 1000, "random"),
    (3, 90, 100, "one"), (3, 90, 500, "two"),
    (3, 300, 2, "random"),             # two buckets: ranks in the hundreds
    (5, 513, 300, "random"),
    (4, 1900, 1024, "random"),         # too much LDS for the projection launch
    (70, 40, 128, "random"),           # more channels than the matrix-core kernel takes
    (3, 60, 4096, "random"),
    (3, 900, 256, "random"),           # lists instead of fold rounds: seven coordinates per bucket
    (3, 260, 64, "random"), (3, 700, 100, "random"),
])
def test_tables(oracle, d, F, D, kind):
    rng = np.random.default_rng(F + D)
    N, L, M = 2, 12, 2
    X = np.cumsum(rng.standard_normal((N, L, d)) * 0.3, axis=1).astype(np.float32)
    W = rng.standard_normal((M, d, F)).astype(np.float32)
    hash_ = {"random": rng.integers(0, D, size=(M, 2 * F)), "one": np.full((M, 2 * F), D - 1),
             "two": rng.integers(0, 2, size=(M, 2 * F)) * (D - 1)}[kind].astype(np.int32)
    sign = (2.0 * rng.integers(0, 2, size=(M, 2 * F)) - 1.0).astype(np.float32)
    got = rfsf.rfsf_ts_features(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), torch.from_numpy(hash_).cuda(),
                                torch.from_numpy(sign).cuda(), 1.5, D).cpu().numpy()
    err = block_errors(got, oracle.features(X, W, hash_, sign, 1.5, D), M, D)
    print(f"d={d} F={F} D={D} {kind}: block errors {err}")
    assert np.all(err <= FP32_BLOCK_TOL)
