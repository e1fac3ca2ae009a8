"""fp16 direct-copy workgroups of three 64-column tiles and of four 64-deep stages: edges of
the tile in every dimension, K of less than a slab, around the length from
which the pipeline runs one slab ahead, and with a remainder.  Small integers:
bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2309_08978_amd as nj
import workloads
from gpu_util import gpu_matmul

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (127, 184, 64), (129, 200, 72), (65, 192, 448), (130, 392, 456), (64, 776, 520)])
@pytest.mark.parametrize("batch", [1, 3])
def test_wide_and_four_stage_tiles(batch, M, N, K):
    A, B = workloads.small_int_operands([batch, M, N, K], batch, M, K, N, "f16")
    R = oracle.matmul(A, B)
    cfgs = [c for c in nj.configs() if c["family"] == "gemm_f16" and c["direct"] == 1
            and (c["name"].endswith("_n3") or (c["Kt"] == 64 and c["stages"] == 4)) and (c["split"] == 1 or c["split"] == 2 and K >= 256)]
    assert len({c["name"] for c in cfgs}) >= 4
    for c in cfgs:
        assert np.array_equal(gpu_matmul(A, B, cfg=c["id"]), R), (c["name"], c["split"])
