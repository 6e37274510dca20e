"""Streaming kernel: a step's factor entries are multiplied with each other before they meet the tensor, so factors whose scales
cancel give the result that they give at scale one.  X, one column mode's factor and another one's are scaled by powers of two
that leave every product of factor entries alone; products of X with one factor alone leave the type's range, above or
below.  Powers of two commute with rounding, so the results agree bit by bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_14891_amd import inputs

pytestmark = pytest.mark.gpu

SCALES = {torch.float32: (83, 50), torch.float64: (700, 500)}       # of X, of a factor: together beyond 2^128, 2^1024
KEYS = {"deep": 1, "small_route": 2, "fuse_bytes": 1, "inner_splits": 1, "target_items": 64, "fuse_rows": 2, "pair_rows": 2, "lead_last": 2}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("col_blocks", [1, 2, 3, 4])
@pytest.mark.parametrize("row_blocks", [1, 2, 3, 4])
def test_scales_that_cancel(row_blocks, col_blocks, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if row_blocks * col_blocks == 16 and dtype == torch.float64:
        pytest.skip("no tile of sixteen fp64 accumulators")
    from paper_2510_14891_amd import binding as mt
    dims, R = (200, 3, 90, 44), 16 * col_blocks - 1
    X = inputs.uniform(3, int(np.prod(dims)), 0.5, 1.0, dtype=dtype).cuda()
    A = [inputs.uniform(40 + m, (I, R), 0.5, 1.0, dtype=dtype).cuda() for m, I in enumerate(dims)]
    ex, ea = SCALES[dtype]
    try:
        for key, value in dict(KEYS, row_blocks=row_blocks).items():
            mt.mttkrp_tune_set(key, value)
        for k in (0, 1):
            plan = mt.mttkrp_plan_describe(dims, R, k, X.element_size())
            print("scales k=%d %s %s" % (k, dtype, plan), flush=True)
            assert "rows_per_wave=%d " % (16 * row_blocks) in plan and "col_blocks=%d " % col_blocks in plan
            assert "inner_mode=2 " in plan and "fused_modes=-1 " in plan and "shape=rows" not in plan
            want = mt.mttkrp_dense(X, dims, A, k).clone()
            assert bool(torch.isfinite(want).all())
            for up, down in ((2, 3), (3, 2)):
                for sign in (1, -1):
                    B = list(A)
                    B[up], B[down] = A[up] * 2.0 ** (sign * ea), A[down] * 2.0 ** (-sign * ea)
                    got = mt.mttkrp_dense(X * 2.0 ** (sign * ex), dims, B, k)
                    assert torch.equal(got * 2.0 ** (-sign * ex), want), (k, up, down, sign)
    finally:
        for key in list(KEYS) + ["row_blocks"]:
            mt.mttkrp_tune_set(key, 0)
