"""The blocked factorisation and solves of CP-ALS at the edges of their tiles: one sweep, every factor against a float64
Cholesky solve on the CPU from the same factors before it.

Ranks around the 4, 16, 32 and 64 columns that the kernels take at a time, row counts around the 16 rows of a workgroup and
the 256 of a short factor, three to eight modes' factors, and ranks beyond two and beyond eight blocks.  Tolerance: both sides solve V a = m backward stably, so each is within a small
multiple of R eps cond(V) of the exact rows (the standard bound of a Cholesky solve); m, a sum of n products of random sign, adds
sqrt(n) eps cond(V)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SHAPES = [((17, 16, 15), R) for R in (1, 3, 4, 5, 15, 16, 17, 31, 33, 63, 64)] + \
         [((33, 17, 40), R) for R in (65, 79, 80, 81, 96, 97, 127, 128, 129, 160, 193)] + \
         [((128, 129, 9), 2), ((255, 256, 7), 8), ((257, 5, 6), 9), ((127, 257, 256), 16), ((2, 90, 1), 2)] + \
         [((4, 3, 5, 3), 11), ((4, 3, 4, 3, 4, 3, 4, 3), 7), ((2, 90, 80), 70), ((16, 50, 40), 257), ((700, 40, 30), 288), ((9000, 24, 20), 130), ((40, 45, 50), 320), ((40, 45, 50), 321), ((40, 45, 50), 545), ((40, 45, 50), 1030)]


@pytest.mark.parametrize("dims,R", SHAPES)
def test_one_sweep_at_tile_edges(dims, R):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    rng = np.random.default_rng(R)
    X = rng.standard_normal(int(np.prod(dims)))
    A0 = [rng.standard_normal((I, R)) for I in dims]
    Ad = [torch.from_numpy(a).cuda() for a in A0]
    print("cp-als blocks dims=%s R=%d" % (dims, R), flush=True)
    mt.mttkrp_cpals(torch.from_numpy(X).cuda(), dims, Ad, 1, 0.0)
    torch.cuda.synchronize()
    got = [a.cpu().numpy() for a in Ad]
    Xn = X.reshape(dims, order="F")
    A = [a.copy() for a in A0]
    for k in range(len(dims)):
        rest = [m for m in range(len(dims)) if m != k]
        krp, V = np.ones((1, R)), np.ones((R, R))
        for m in rest:
            krp = (krp[:, None, :] * A[m][None, :, :]).reshape(-1, R)
            V *= A[m].T @ A[m]
        M = np.transpose(Xn, [k] + rest).reshape(dims[k], -1) @ krp
        want = np.linalg.solve(V, M.T).T
        norm = np.linalg.norm(want, axis=0)
        want /= np.where(norm > 0, norm, 1.0)
        bound = (4.0 * R + np.sqrt(krp.shape[0])) * np.finfo(np.float64).eps * np.linalg.cond(V)
        err = np.linalg.norm(got[k] - want) / np.linalg.norm(want)
        assert err <= bound, (k, err, bound)
        A[k] = got[k]                     # the next mode starts from what the driver has
