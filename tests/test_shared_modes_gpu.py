"""A mode's result from the shared sweep's intermediate where its work is cut: rows with few pairs (a thread a row and one or four
columns, R at which groups of columns overlap, the sizes around the line to a workgroup a row), and many segments (seventeen, the fewest
that 64 threads add, and more than eight for each of them).  Against matrix products in fp64; tolerances are those of every parity test: 1e-12
(fp64) and 1e-5 (fp32), normwise."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_14891_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [((5, 4, 3, 16384, 3), 4), ((5, 4, 3, 16383, 3), 4), ((5, 4, 3, 5500, 3), 3), ((5, 4, 3, 9001, 2), 7), ((3, 7001, 2, 5, 4), 18),
         ((2, 17000, 2, 16, 8, 2), 5), ((60, 241, 1100), 5), ((4, 4, 4, 20011, 4), 4), ((3, 40009, 3, 5), 10)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dims,R", CASES)
def test_modes_of_a_shared_sweep(dims, R, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    X = inputs.uniform(7, int(np.prod(dims)), -1.0, 1.0, dtype=dtype)
    A = [inputs.uniform(70 + m, (I, R), -1.0, 1.0, dtype=dtype) for m, I in enumerate(dims)]
    print("shared modes dims=%s R=%d" % (dims, R), flush=True)
    got = mt.mttkrp_dense_all_modes_shared(X.cuda(), dims, [a.cuda() for a in A])
    X64, A64 = X.numpy().astype(np.float64), [a.numpy().astype(np.float64) for a in A]
    for k, M in enumerate(got):
        low, high = np.ones((1, R)), np.ones((1, R))
        for a in A64[:k]:
            low = (a[:, None, :] * low[None]).reshape(-1, R)
        for a in A64[k + 1:]:
            high = (a[:, None, :] * high[None]).reshape(-1, R)
        part = (X64.reshape(-1, low.shape[0]) @ low).reshape(high.shape[0], dims[k], R)
        want = (part * high[:, None, :]).sum(0)
        err = np.linalg.norm(M.cpu().numpy() - want) / np.linalg.norm(want)
        assert err <= (1e-12 if dtype == torch.float64 else 1e-5), (k, err)
