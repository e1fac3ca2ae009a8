"""Products whose operands no 16-byte-load configuration can run, and products
of single rows: odd sizes, odd leading dimensions, base pointers off by one
element, the padding between rows and slices filled with NaN.  Small integers:
bit-exact against the oracle, through the default configuration and through
every configuration that takes any alignment."""
import numpy as np
import pytest

import oracle
import paper_2309_08978_amd as nj
import workloads
from gpu_util import dtype_code, host

pytestmark = pytest.mark.gpu

# batch, M, N, K: the branches of the predefined choice and the edges of the
# kernels (tile remainders, K of less than a slab, of whole slabs and more; N
# of less than one load and just past one; rows per slot below and past U)
TILES = [(12, 31, 31, 64), (12, 31, 64, 31), (5, 77, 77, 64), (5, 77, 64, 77), (3, 129, 131, 97), (16, 257, 259, 33),
         (70, 128, 129, 40), (2, 65, 3, 7), (2, 3, 5, 1), (1, 333, 517, 203), (1, 70, 1001, 1025)]
ROWS = [(3, 1, 5, 9), (2, 1, 1, 1), (4, 1, 8, 64), (4, 1, 9, 65), (6, 1, 1023, 128), (6, 1, 64, 511), (5, 1, 130, 129),
        (5, 1, 127, 256), (3, 1, 128, 1025), (2, 1, 33, 2049), (2, 1, 7, 0)]


def _operand(x, pad, shift):
    """x [batch, rows, cols] on the GPU with a leading dimension of cols + pad,
    a NaN-filled gap of 3 elements between slices, beginning `shift` elements
    into its buffer.  Returns (buffer, pointer, ld, stride)."""
    import torch
    b, r, c = x.shape
    ld = max(1, c + pad)
    stride = max(1, r * ld + 3)
    t = torch.float16 if x.dtype == np.float16 else torch.float32
    # the buffer ends with the last element of the last row
    buf = torch.full((shift + (b - 1) * stride + max(0, r - 1) * ld + c,), float("nan"), dtype=t, device="cuda:0")
    if x.size:
        idx = shift + (np.arange(b)[:, None, None] * stride + np.arange(r)[None, :, None] * ld + np.arange(c)[None, None, :])
        buf[torch.from_numpy(idx.reshape(-1)).to("cuda:0")] = torch.from_numpy(x.reshape(-1)).to("cuda:0")
    return buf, buf.data_ptr() + shift * buf.element_size(), ld, stride


def _check(batch, M, N, K, dt, pads, shifts, configs):
    import torch
    A, B = workloads.small_int_operands([batch, M, N, K], batch, M, K, N, dt)
    A, B = A.reshape(batch, M, K), B.reshape(batch, K, N)
    R = oracle.matmul(A, B).reshape(batch, M, N) if K else np.zeros((batch, M, N))
    keepA, pA, lda, sA = _operand(A, pads[0], shifts[0])
    keepB, pB, ldb, sB = _operand(B, pads[1], shifts[1])
    ldc, sC = N + pads[2], M * (N + pads[2]) + 1
    for cfg in configs:
        C = torch.full((batch * sC,), 7.5, dtype=torch.float32, device="cuda:0")
        if cfg is None:
            rc = nj.nnjit_batched_matmul(batch, M, N, K, pA, lda, sA, pB, ldb, sB, C, ldc, sC, dtype_code(dt))
        else:
            rc = nj.nnjit_matmul_config(cfg["id"], batch, M, N, K, pA, lda, sA, pB, ldb, sB, C, ldc, sC, dtype_code(dt))
        what = "default" if cfg is None else (cfg["name"], cfg["split"])
        assert rc == 0, (what, nj.nnjit_last_error())
        got = host(C).reshape(batch, sC)
        rows = got[:, :M * ldc].reshape(batch, M, ldc)
        assert np.array_equal(rows[:, :, :N], R), what
        assert np.all(rows[:, :, N:] == 7.5) and np.all(got[:, M * ldc:] == 7.5), (what, "wrote outside C")
    del keepA, keepB


def _any_alignment(dt, rows):
    return [c for c in nj.configs() if c["family"] == "gemm_" + dt and c["vec"] < 16 and c["split"] in (1, 4)
            and (c["Mt"] == 1) == rows]


@pytest.mark.parametrize("dt", ["f32", "f16"])
@pytest.mark.parametrize("shape", TILES + ROWS)
def test_any_alignment(dt, shape):
    batch, M, N, K = shape
    cfgs = [None] + [c for c in _any_alignment(dt, M == 1) if c["split"] == 1 or K >= 8 * c["Kt"]]
    for pads, shifts in (((0, 0, 0), (0, 0)), ((1, 3, 1), (1, 0)), ((0, 6, 2), (0, 3))):
        _check(batch, M, N, K, dt, pads, shifts, cfgs)


@pytest.mark.parametrize("dt", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(64, 256, 256, 64), (12, 200, 200, 64), (12, 200, 64, 200), (1, 64, 768, 768),
                                   (1, 520, 512, 1032), (1, 1024, 4096, 64), (300, 128, 128, 16), (4, 1, 512, 128)])
def test_predefined_aligned(dt, shape):
    """The predefined configurations of aligned shapes, and of the same shapes
    with misaligned operands."""
    batch, M, N, K = shape
    _check(batch, M, N, K, dt, (0, 0, 0), (0, 0), [None])
    _check(batch, M, N, K, dt, (0, 0, 0), (1, 1), [None])


# the predefined choice for single rows: every segment width, the split, and its
# neighbours at either end
@pytest.mark.parametrize("dt", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(8, 1, 128, 4096), (8, 1, 128, 4095), (8, 1, 127, 4096), (8, 1, 64, 4096), (2, 1, 1032, 2048),
                                   (257, 1, 264, 40), (257, 1, 130, 136), (130, 1, 1032, 24), (600, 1, 72, 520),
                                   (2, 1, 8200, 264), (3, 1, 2056, 300)])
def test_predefined_single_rows(dt, shape):
    batch, M, N, K = shape
    _check(batch, M, N, K, dt, (0, 0, 0), (0, 0), [None])
    _check(batch, M, N, K, dt, (0, 0, 0), (1, 1), [None])
    _check(batch, M, N, K, dt, (0, 3, 1), (0, 0), [None])


# long sums over few tiles (split where a split served them before, and the
# lengths and tile counts around that), up to 16 rows over few and many columns
@pytest.mark.parametrize("dt", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(1, 39, 1264, 5072), (1, 40, 1256, 1016), (8, 16, 128, 4096), (1, 256, 256, 4096),
                                   (1, 33, 513, 8193), (8, 23, 53, 1621), (1, 16, 4096, 1024), (1, 16, 8200, 1032),
                                   (1, 9, 8192, 40), (1, 14, 2584, 2064), (32, 7, 1032, 72)])
def test_predefined_long_sums_and_few_rows(dt, shape):
    batch, M, N, K = shape
    _check(batch, M, N, K, dt, (0, 0, 0), (0, 0), [None])
    _check(batch, M, N, K, dt, (0, 0, 0), (1, 1), [None])


def _captured(batch, M, N, K, dt, shift):
    """The default call under capture on a stream that has run nothing before:
    the return code, and whether two replays give the product."""
    import torch
    A, B = workloads.small_int_operands([batch, M, N, K], batch, M, K, N, dt)
    A, B = A.reshape(batch, M, K), B.reshape(batch, K, N)
    R = oracle.matmul(A, B).reshape(batch, M, N)
    keepA, pA, lda, sA = _operand(A, 0, shift)
    keepB, pB, ldb, sB = _operand(B, 0, shift)
    if not shift:   # slices without a gap, so that the operands are aligned
        keepA, keepB = (torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0") for x in (A, B))
        pA, lda, sA, pB, ldb, sB = keepA.data_ptr(), K, M * K, keepB.data_ptr(), N, K * N
    C = torch.zeros((batch, M, N), dtype=torch.float32, device="cuda:0")
    call = lambda st: nj.nnjit_batched_matmul(batch, M, N, K, pA, lda, sA, pB, ldb, sB, C.data_ptr(), N, M * N,
                                              dtype_code(dt), st)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        rc = call(stream)
    for _ in range(2 if rc == 0 else 0):
        C.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        assert np.array_equal(host(C).reshape(batch, M, N), R)
    return rc


@pytest.mark.parametrize("dt", ["f32", "f16"])
def test_predefined_split_takes_scratch_only_where_it_did(dt):
    """A split needs scratch, which a stream under capture cannot get: misaligned
    operands and shapes that a split never served run under capture at once."""
    assert _captured(8, 1, 128, 4096, dt, 1) == 0      # misaligned operands of a split shape
    assert _captured(2, 1, 64, 8192, dt, 0) == 0       # too few columns for a split before
    assert _captured(8, 1, 128, 4095, dt, 0) == 0      # a shape of any alignment
    assert _captured(8, 16, 128, 4096, dt, 1) == 0
    assert _captured(1, 40, 72, 8192, dt, 0) == 0      # more splits than there are would be needed
    assert _captured(8, 1, 128, 4096, dt, 0) == nj.NNJIT_EHIP
    assert "capture" in nj.nnjit_last_error()


def test_binding_views_and_refusals_on_the_gpu():
    """The tensor conveniences on operands that take the short checks and on
    ones that need the full ones: views with padded rows, one-row and expanded
    batches, empty products; and what is refused stays refused."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    big = torch.randint(-8, 9, (4, 40, 64), generator=g, device="cuda").float()
    W = torch.randint(-8, 9, (4, 64, 48), generator=g, device="cuda").float()

    def same(C, R):
        return bool((C.double() == R).all())

    for A, B in ((big[0], W[0]), (big[0, :, :30], W[0, :30, :17]), (big[0, 3:4], W[0]), (big[0, ::2], W[0]),
                 (big[0, :1, :1], W[0, :1, :1])):
        assert same(nj.matmul(A, B), A.double() @ B.double())
    for A, B in ((big, W), (big[:, 1:2], W), (big[:, :, 5:30], W[:, 5:30, 1:]), (big[:1].expand(4, 40, 64), W),
                 (big[1:2], W[1:2]), (big[::2], W[::2])):
        R = torch.bmm(A.double().contiguous(), B.double().contiguous())
        assert same(nj.batched_matmul(A, B), R)
        C = torch.full((R.shape[0], R.shape[1] + 1, R.shape[2] + 3), 9.0, device="cuda")
        nj.batched_matmul(A, B, C[:, :R.shape[1], :R.shape[2]])
        assert same(C[:, :R.shape[1], :R.shape[2]], R) and bool((C[:, R.shape[1]:] == 9).all())
    assert nj.matmul(big[0, :0], W[0]).shape == (0, 48)
    assert bool((nj.matmul(big[0, :, :0], W[0, :0]) == 0).all())
    bad = [(ValueError, lambda: nj.matmul(big[0], W[0].t())), (ValueError, lambda: nj.matmul(big[0].t(), big[0])),
           (TypeError, lambda: nj.matmul(big[0], W[0].half())), (ValueError, lambda: nj.matmul(big[0], W[0].cpu())),
           (ValueError, lambda: nj.matmul(big[0], W[0, :63])),
           (ValueError, lambda: nj.matmul(big[0, :1].expand(40, 64), W[0])),
           (TypeError, lambda: nj.matmul(big[0], W[0], torch.empty(40, 48, device="cuda", dtype=torch.float16))),
           (ValueError, lambda: nj.matmul(big[0], W[0], torch.empty(1, 40, 48, device="cuda"))),
           (ValueError, lambda: nj.batched_matmul(big, W, torch.empty(1, 40, 48, device="cuda").expand(4, 40, 48))),
           (ValueError, lambda: nj.batched_matmul(big, W[:3])),
           (TypeError, lambda: nj.matmul(big[0].double(), W[0].double()))]
    for exc, call in bad:
        with pytest.raises(exc):
            call()
