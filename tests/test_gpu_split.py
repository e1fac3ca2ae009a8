"""fp32 products on the bf16 matrix cores (operands split in three bf16 parts):
what the split does not serve -- operands that are not finite, that round to a
bf16 infinity, sums that overflow, operands whose last bits are below the
smallest bf16 subnormal -- comes out as fp32 arithmetic gives it."""
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


def _bound(A, B):
    K = A.shape[1]
    return (K + 4) * 2.0 ** -24 * (np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)) + K * 2.0 ** -148


@pytest.mark.parametrize("M,N,K", SHAPES + [(300, 520, 72)])
@pytest.mark.parametrize("a,b", [(1e-37, 1e36), (1e-36, 1e30), (1e-34, 1e25), (1e-39, 1e36), (3e-41, 1.0), (1e-37, 1e14),
                                 (1e-39, 4e9), (1e-40, 3e17)])
def test_tiny_operands_that_meet_large_ones(M, N, K, a, b):
    """Tiny operands times large ones, in either order, whole or in one row and
    one column beside ordinary ones: the same bound as above, also where the
    sums are not small."""
    rng = np.random.default_rng(14)
    A0 = rng.uniform(0.5, 1, (M, K)).astype(np.float32) * rng.choice([-1, 1], (M, K)).astype(np.float32)
    B0 = rng.uniform(0.5, 1, (K, N)).astype(np.float32) * rng.choice([-1, 1], (K, N)).astype(np.float32)
    few_a, few_b = A0.copy(), B0.copy()
    few_a[17, 5:] *= np.float32(a)      # a row [1, a, ...] meets a column [1, b, ...]
    few_b[5:, N - 2] *= np.float32(b)
    whole_a, whole_b = A0 * np.float32(a), B0 * np.float32(b)
    for A, B in ((whole_a, whole_b), (few_a, few_b), (few_a, whole_b)):
        for X, Y in ((A, B), (np.ascontiguousarray(B.T), np.ascontiguousarray(A.T))):
            R = X.astype(np.float64) @ Y.astype(np.float64)
            bound = _bound(X, Y)
            for c in _configs():
                if c["vec"] < 16 or Y.shape[1] % 4 == 0:
                    assert np.all(np.abs(_run(c, X, Y) - R) <= bound), (c["name"], c["split"])


@pytest.mark.parametrize("M,N,K", SHAPES + [(300, 520, 72)])
def test_a_single_tiny_operand_at_any_place(M, N, K):
    """Row r of A (and column r of B) is zero but for one tiny value, none of
    them the first of the eight that are split together."""
    rng = np.random.default_rng(17)
    at = lambda n: 8 * (np.arange(n) % (K // 8)) + 1 + np.arange(n) % 7
    A, B = np.zeros((M, K), np.float32), rng.uniform(0.5, 1, (K, N)).astype(np.float32)
    A[np.arange(M), at(M)] = (rng.uniform(1, 2, M) * 2.0 ** rng.integers(-140, -110, M)).astype(np.float32)
    At, Bt = rng.uniform(0.5, 1, (M, K)).astype(np.float32), np.zeros((K, N), np.float32)
    Bt[at(N), np.arange(N)] = (rng.uniform(1, 2, N) * 2.0 ** rng.integers(-140, -110, N)).astype(np.float32)
    for X, Y in ((A, B), (At, Bt)):
        R = X.astype(np.float64) @ Y.astype(np.float64)
        for c in _configs():
            assert np.all(np.abs(_run(c, X, Y) - R) <= 2.0 ** -24 * np.abs(R) * 2 + 2.0 ** -149), (c["name"], c["split"])


@pytest.mark.parametrize("lo", [2.0 ** -110, 2.0 ** -106, 2.0 ** -103])
def test_operands_at_the_limit_of_the_split(lo):
    """Every operand of A in [lo, 8 lo): at and above 2^-110 the three parts
    hold all bits (the low ones as bf16 subnormals), so the sums, all far below
    the test of small sums, are right without it."""
    M, N, K = SHAPES[1]
    rng = np.random.default_rng(15)
    A = (rng.uniform(1, 8, (M, K)) * lo).astype(np.float32)
    B = rng.uniform(0.5, 1, (K, N)).astype(np.float32)
    R = A.astype(np.float64) @ B.astype(np.float64)
    for c in _configs():
        assert np.all(np.abs(_run(c, A, B) - R) <= _bound(A, B)), (c["name"], c["split"])


@pytest.mark.parametrize("M,N,K", SHAPES + [(300, 520, 72)])
def test_only_the_sums_concerned_are_taken_anew(M, N, K):
    """Rows of weights of which one is tiny, rows and columns of zeros, a row
    that overflows: every other sum keeps its bits."""
    rng = np.random.default_rng(16)
    A = rng.uniform(0.5, 1, (M, K)).astype(np.float32)
    B = rng.standard_normal((K, N), dtype=np.float32)
    X, Y = A.copy(), B.copy()
    X[3, 2], X[40, K - 1] = 1e-35, 1e-40
    X[5], X[33] = 0.0, 0.0
    X[64] = 3.3e38
    Y[:, 7] = 0.0
    rows = np.setdiff1d(np.arange(M), [3, 40, 5, 33, 64])
    cols = np.setdiff1d(np.arange(N), [7])
    for c in _configs():
        want, C = _run(c, A, B), _run(c, X, Y)
        assert np.array_equal(C[np.ix_(rows, cols)], want[np.ix_(rows, cols)]), (c["name"], c["split"])
        assert not C[[5, 33]].any() and not C[rows][:, 7].any() and not C[[3, 40], 7].any(), (c["name"], c["split"])
        R = X[[3, 40]].astype(np.float64) @ Y.astype(np.float64)
        assert np.all(np.abs(C[[3, 40]] - R) <= _bound(X[[3, 40]], Y)), (c["name"], c["split"])


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


@pytest.mark.parametrize("K", [8, 40, 200, 1024])
@pytest.mark.parametrize("value", [1.0038986, 1.0, 1.9999999, 0.7])
def test_equal_operands(K, value):
    """The dropped part products of equal operands have one sign: up to 2^-24 of
    each product (1.0038986 comes nearest), besides one rounding per part
    product and 16 k, and those of the sums over waves and splits."""
    M, N = 72, 136
    v = np.float32(value)
    A, B = np.full((M, K), v), np.full((K, N), v)
    R = K * float(v) * float(v)
    for c in _configs():
        C = _run(c, A, B)
        assert np.all(np.abs(C - R) <= (1 + 6 * -(-K // 16) + 8) * 2.0 ** -24 * R), (c["name"], c["split"])


@pytest.mark.parametrize("M,N,K", [(100, 768, 256), (33, 200, 40), (300, 264, 72)])
def test_rows_past_the_end_are_not_looked_into(M, N, K):
    """Tiles that reach past M and N: what is read for the rows and columns
    outside changes no bit of the sums inside, whatever lies in the first row
    and behind the operands."""
    rng = np.random.default_rng(18)
    A = rng.standard_normal((M, K), dtype=np.float32)
    B = rng.standard_normal((K, N), dtype=np.float32)
    X = A.copy()
    X[0] = 0.0
    for c in _configs():
        if c["split"] == 1:
            want, C = _run(c, A, B), _run(c, X, B)
            assert np.array_equal(C[1:], want[1:]) and not C[0].any(), c["name"]
