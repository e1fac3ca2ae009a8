"""fp32 products on the bf16 matrix cores (operands split in three bf16 parts):
what the split does not serve -- operands that are not finite, that round to a
bf16 infinity, sums that overflow, operands whose low parts are subnormal --
comes out as fp32 arithmetic gives it."""
import numpy as np
import pytest

import paper_2309_08978_amd as nj
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

# K: a short tail slab only, whole slabs in the unchecked loop and a tail
SHAPES = [(70, 136, 40), (100, 264, 200)]


def _configs():
    return [c for c in nj.configs() if c["family"] == "gemm_f32" and c["direct"] == 2 and c["split"] in (1, 2)]


def _run(c, A, B):
    import torch
    C = torch.full((A.shape[0], B.shape[1]), 7.0, dtype=torch.float32, device="cuda:0")
    nj.matmul(dev(A), dev(B), C, cfg=c["id"])
    return host(C).astype(np.float64)


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_not_finite_operands_and_sums(M, N, K):
    rng = np.random.default_rng(11)
    A = rng.standard_normal((M, K), dtype=np.float32)
    B = rng.standard_normal((K, N), dtype=np.float32)
    A[3, 5], A[M - 1, K - 1], A[9, 0], A[9, 3] = np.inf, np.nan, -np.inf, np.inf
    B[7, 8], B[5, N - 1] = 3.4e38, -np.inf          # 3.4e38 rounds to a bf16 infinity
    A[:, 7] = np.where(np.arange(M) % 2, 0.25, 4.0)  # times 3.4e38: finite or overflowing
    with np.errstate(all="ignore"):
        R = A.astype(np.float64) @ B.astype(np.float64)
        R = np.where(np.abs(R) > 3.5e38, np.copysign(np.inf, R), R)
    for c in _configs():
        C = _run(c, A, B)
        assert np.array_equal(np.isnan(C), np.isnan(R)), c["name"]
        assert np.array_equal(np.isinf(C), np.isinf(R)) and np.array_equal(C[np.isinf(R)], R[np.isinf(R)]), c["name"]
        fin = np.isfinite(R)
        small = fin & (np.abs(R) < 1e30)
        assert np.all(np.abs(C[small] - R[small]) <= 2e-6 * K * 25), c["name"]
        assert np.allclose(C[fin & ~small], R[fin & ~small], rtol=1e-5), c["name"]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("scale", [1e-30, 1e-34, 1e-36, 2e-38])
def test_tiny_operands_keep_fp32_precision(M, N, K, scale):
    """A scaled by a tiny factor, whole or in one row.  A summation order's
    error is at most gamma(K) sum |a b|; each fp32 result may also be off by
    the smallest subnormal per term."""
    rng = np.random.default_rng(12)
    A = rng.standard_normal((M, K), dtype=np.float32)
    B = rng.standard_normal((K, N), dtype=np.float32)
    whole = (A * np.float32(scale)).astype(np.float32)
    row = A.copy()
    row[17] *= np.float32(scale)
    for X in (whole, row):
        R = X.astype(np.float64) @ B.astype(np.float64)
        bound = (K + 4) * 2.0 ** -24 * (np.abs(X).astype(np.float64) @ np.abs(B).astype(np.float64)) + K * 2.0 ** -148
        for c in _configs():
            if c["vec"] == 16 or c["split"] == 1:
                assert np.all(np.abs(_run(c, X, B) - R) <= bound), (c["name"], c["split"])


@pytest.mark.parametrize("K", [4, 16, 20, 32, 36, 48])
def test_zero_sums_leave_the_other_rows_alone(K):
    """K of one to three slabs: staging registers that no slab was loaded into
    are not operands, so a row of zero sums changes no bit of the other rows
    (a wave that takes its sums anew rounds them otherwise)."""
    M, N = 300, 264
    rng = np.random.default_rng(13)
    A = rng.standard_normal((M, K), dtype=np.float32)
    B = rng.standard_normal((K, N), dtype=np.float32)
    Z = A.copy()
    Z[::32] = 0.0
    keep = np.arange(M) % 32 != 0
    for c in _configs():
        if c["split"] == 1:
            want = _run(c, A, B)
            for _ in range(3):
                C = _run(c, Z, B)
                assert np.array_equal(C[keep], want[keep]) and not C[~keep].any(), c["name"]
