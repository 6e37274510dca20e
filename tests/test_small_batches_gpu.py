"""The kernel for small tensors where its batches and its rows end: columns of one to nine steps of four (a remainder runs in a batch
of a quarter, a half, three quarters of the full one), rows that are not a multiple of the two or four consecutive ones a lane
holds, one to six column modes and none, one to four blocks of output columns, against float64 sums on the CPU.

Tolerance, entry by entry: n terms of d factors each, added in any order, are within (n + d) eps times the sum of the terms' absolute
values of the exact sum (the standard bound); the reference, in 64 bits, adds its own (n + d) eps of that type."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CASES = [((35, 3, c), 10, 1) for c in (1, 4, 5, 9, 13, 16, 17, 21, 25, 29, 32, 33, 36)] + \
        [((m, 5, 9), 12, 1) for m in (17, 33, 34, 37, 38, 39, 63, 66, 129)] + \
        [((37, c, 6), R, 2) for c, R in ((3, 31), (9, 32), (13, 48), (18, 40), (7, 64), (19, 50), (11, 70))] + \
        [((35, c, 2), R, 0) for c, R in ((1, 4), (9, 17), (15, 33), (21, 64), (70, 49))] + \
        [((17, 3, 2, 3, 5), 9, k) for k in range(5)] + [((5, 3, 2, 3, 2, 4), 20, k) for k in (0, 3)] + \
        [((6, 2, 3, 2, 3, 2, 3), 33, k) for k in (0, 6)] + [((19, 1, 3, 1, 2, 1), 7, k) for k in (0, 2)] + [((21, 18), 30, 1)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("groups", [1, 4])
@pytest.mark.parametrize("dims,R,k", CASES)
def test_batches_and_rows_at_their_ends(dims, R, k, groups, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    rng = np.random.default_rng(R + sum(dims))
    X = torch.from_numpy(rng.standard_normal(int(np.prod(dims)))).to(dtype)
    A = [torch.from_numpy(rng.standard_normal((I, R))).to(dtype) for I in dims]
    print("small batches dims=%s R=%d k=%d groups=%d %s" % (dims, R, k, groups, dtype), flush=True)
    mt.mttkrp_tune_set("small_route", 1)
    mt.mttkrp_tune_set("small_groups", groups)
    try:
        assert "small_route=1" in mt.mttkrp_plan_describe(dims, R, k, X.element_size())
        got = mt.mttkrp_dense(X.cuda(), dims, [a.cuda() for a in A], k).cpu().numpy().astype(np.float64)
    finally:
        mt.mttkrp_tune_set("small_route", 0)
        mt.mttkrp_tune_set("small_groups", 0)
    rest = [m for m in range(len(dims)) if m != k]
    krp = np.ones((1, R))
    for m in rest:
        krp = (krp[:, None, :] * A[m].numpy().astype(np.float64)[None, :, :]).reshape(-1, R)
    Xk = np.transpose(X.numpy().astype(np.float64).reshape(dims, order="F"), [k] + rest).reshape(dims[k], -1)
    want, size = Xk @ krp, np.abs(Xk) @ np.abs(krp)
    eps = np.finfo(np.float64 if dtype == torch.float64 else np.float32).eps + np.finfo(np.float64).eps
    bound = (krp.shape[0] + len(dims)) * eps * size
    assert (np.abs(got - want) <= bound).all(), np.max(np.abs(got - want) / np.maximum(bound, 1e-300))
