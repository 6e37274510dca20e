"""The update of a factor where its work is cut: one sweep, the last factor, its weights and the sweep's fit against
float64 on the CPU from the same factors before it.

The ranks are those of one to four blocks of 16 columns; the rows those around one tile, one round of the workgroup's wavefronts,
what stays in one workgroup's LDS (880, 432, 304 and 208 rows) and the first size of two launches, and several rounds of
many workgroups.  Above rank 64 the ranks at which four, eight and sixteen wavefronts share a solve and the first beyond.  Tolerance: both sides solve V a = m backward stably, so each is within a small multiple of R eps cond(V) of the exact
rows; m, a sum of n products of random sign, adds sqrt(n) eps cond(V)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CASES = [(R, I) for R, rows in ((10, (257, 880, 881, 1025, 40000)), (17, (15, 256, 257, 432, 433)), (32, (16, 432, 433, 20000)),
                                (33, (128, 129, 304, 305)), (48, (304, 305, 5000)), (49, (5, 127, 208, 209)), (64, (129, 208, 209, 18000)),
                                (65, (33,)), (128, (16, 100)), (129, (17,)), (256, (15, 31)), (257, (48,)), (512, (33,)), (513, (15,)))
         for I in rows]


@pytest.mark.parametrize("R,I", CASES)
def test_update_of_the_last_factor(R, I):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    dims = (12, 11, I) if R <= 64 else (40, 45, I)
    rng = np.random.default_rng(1000 * R + I)
    X = rng.standard_normal(int(np.prod(dims)))
    Ad = [torch.from_numpy(rng.standard_normal((n, R))).cuda() for n in dims]
    print("cp-als update dims=%s R=%d" % (dims, R), flush=True)
    lam, fits = mt.mttkrp_cpals(torch.from_numpy(X).cuda(), dims, Ad, 1, 0.0)
    torch.cuda.synchronize()
    A, lam = [a.cpu().numpy() for a in Ad], lam.cpu().numpy()
    krp = (A[1][:, None, :] * A[0][None, :, :]).reshape(-1, R)          # the first index fastest
    M = X.reshape(I, -1) @ krp
    G = [a.T @ a for a in A]
    V = G[0] * G[1]
    want = np.linalg.solve(V, M.T).T
    norm = np.linalg.norm(want, axis=0)
    bound = (4.0 * R + np.sqrt(krp.shape[0])) * np.finfo(np.float64).eps * np.linalg.cond(V)
    assert np.linalg.norm(lam - norm) <= bound * np.linalg.norm(norm)
    want /= norm
    assert np.linalg.norm(A[2] - want) <= bound * np.linalg.norm(want)
    # the fit, from the factors as they are: its terms are sums of R columns and R^2 entries
    norm2 = float(X @ X)
    resid2 = max(norm2 + lam @ (V * G[2]) @ lam - 2.0 * float(lam @ (M * A[2]).sum(0)), 0.0)
    fit = 1.0 - np.sqrt(resid2) / np.sqrt(norm2)
    assert abs(fits[0] - fit) <= 64.0 * R * np.finfo(np.float64).eps * np.sqrt(np.linalg.cond(V)) + 1e-12
