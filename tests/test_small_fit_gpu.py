"""Calls that the newer fit gives to the kernel for small tensors, against the general plan and against matrix products in fp64: two to
eight modes, each number of column modes, the last size that the fit decides (7/8 of 2^20 values) and the first beyond, outputs of several chunks of
columns.  Tolerances are those of every parity test: 1e-12 (fp64) and 1e-5 (fp32), normwise."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_14891_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [((152, 8), 65), ((1868, 257), 13), ((48, 40, 36), 3), ((128, 128, 56), 16), ((128, 128, 57), 16), ((17, 37, 45, 19), 36),
         ((9, 11, 10, 7, 15), 33), ((8, 8, 8, 16, 8, 8), 7), ((7, 9, 10, 7, 7, 17), 38), ((4, 3, 5, 4, 3, 4, 5, 3), 100)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dims,R", CASES)
def test_both_routes_agree(dims, R, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    X = inputs.uniform(5, int(np.prod(dims)), -1.0, 1.0, dtype=dtype)
    A = [inputs.uniform(50 + m, (I, R), -1.0, 1.0, dtype=dtype) for m, I in enumerate(dims)]
    Xd, Ad = X.cuda(), [a.cuda() for a in A]
    X64, A64 = X.numpy().astype(np.float64), [a.numpy().astype(np.float64) for a in A]
    for k in range(len(dims)):
        print("small fit dims=%s R=%d k=%d" % (dims, R, k), flush=True)
        got = mt.mttkrp_dense(Xd, dims, Ad, k)
        mt.mttkrp_tune_set("small_route", 2)
        try:
            general = mt.mttkrp_dense(Xd, dims, Ad, k)
        finally:
            mt.mttkrp_tune_set("small_route", 0)
        low, high = np.ones((1, R)), np.ones((1, R))
        for a in A64[:k]:
            low = (a[:, None, :] * low[None]).reshape(-1, R)
        for a in A64[k + 1:]:
            high = (a[:, None, :] * high[None]).reshape(-1, R)
        want = ((X64.reshape(-1, low.shape[0]) @ low).reshape(high.shape[0], dims[k], R) * high[:, None, :]).sum(0)
        for M in (got, general):
            assert np.linalg.norm(M.cpu().numpy() - want) <= tol * np.linalg.norm(want), (k, M is got)
