"""GPU parity of the CP-ALS driver and the all-modes sweep (include/mttkrp_cpals.h)
against the CPU oracles, through the C ABI.

The driver and the oracle start from the same seeded tensor and initial factors
and take the same steps (see the header), so after a fixed number of sweeps the
fits, the weights and the factors must agree to rounding.  ALS amplifies
rounding differences slowly, so a handful of sweeps is compared at 1e-9, far
inside what a wrong step (a transposed solve, a missing Gram update, a wrong
norm) would produce.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_14891_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding
    binding.lib()
    return binding


def problem(dims, R, seed, rank_true=None, noise=0.0):
    n = int(np.prod(dims))
    if rank_true is None:
        X = inputs.normal(seed, n, 0.0, 1.0)
    else:
        from oracle import cp_als_oracle
        U = [inputs.normal(seed + 50 + m, (I, rank_true), 0.0, 1.0).numpy() for m, I in enumerate(dims)]
        Xn = cp_als_oracle.reconstruct(U, np.ones(rank_true))
        Xn = Xn + noise * inputs.as_ndarray_view(inputs.normal(seed, n, 0.0, 1.0), dims)
        X = torch.from_numpy(np.ascontiguousarray(Xn.reshape(-1, order="F")))
    A0 = [inputs.uniform(seed + 100 + m, (I, R), 0.0, 1.0) for m, I in enumerate(dims)]
    return X, A0


CASES = [((40, 30, 20), 5, 11), ((17, 9, 6, 5), 3, 12), ((33, 20), 4, 13), ((24, 18, 10), 16, 14),
         ((70, 5, 9), 1, 15)]


@pytest.mark.parametrize("dims,R,seed", CASES)
def test_cpals_matches_the_oracle(mt, dims, R, seed):
    from oracle import cp_als_oracle, mttkrp_oracle
    mttkrp_oracle.build()
    X, A0 = problem(dims, R, seed)
    sweeps = 5
    A_ref, lam_ref, fits_ref = cp_als_oracle.cp_als(inputs.as_ndarray_view(X, dims), [a.numpy() for a in A0], sweeps, 0.0)
    Xd = X.cuda()
    Ad = [a.clone().cuda() for a in A0]
    print("cp-als case dims=%s R=%d" % (dims, R), flush=True)
    lam, fits = mt.mttkrp_cpals(Xd, dims, Ad, sweeps, 0.0)
    torch.cuda.synchronize()
    assert len(fits) == sweeps == len(fits_ref)
    np.testing.assert_allclose(fits, fits_ref, rtol=0, atol=1e-10)
    np.testing.assert_allclose(lam.cpu().numpy(), lam_ref, rtol=1e-9)
    for m in range(len(dims)):
        got = Ad[m].cpu().numpy()
        err = np.linalg.norm(got - A_ref[m]) / np.linalg.norm(A_ref[m])
        assert err <= 1e-9, (m, err)


# Ranks above 64 take the blocked Gram / Cholesky / triangular-solve kernels (32 columns at a
# time): just above the switch, a multiple of the block, partial last blocks, a short mode.
LARGE_RANK = [((100, 70, 66), 65, 31), ((120, 110, 100), 96, 32), ((90, 85, 80), 80, 33), ((72, 71, 70, 5), 70, 34),
              ((40, 150, 140), 130, 35)]


@pytest.mark.parametrize("dims,R,seed", LARGE_RANK)
@pytest.mark.parametrize("shared", [False, True])
def test_cpals_large_rank_matches_the_oracle(mt, dims, R, seed, shared):
    from oracle import cp_als_oracle, mttkrp_oracle
    mttkrp_oracle.build()
    X, A0 = problem(dims, R, seed)
    sweeps = 3
    A_ref, lam_ref, fits_ref = cp_als_oracle.cp_als(inputs.as_ndarray_view(X, dims), [a.numpy() for a in A0], sweeps, 0.0)
    Ad = [a.clone().cuda() for a in A0]
    print("cp-als large rank dims=%s R=%d shared=%s" % (dims, R, shared), flush=True)
    lam, fits = mt.mttkrp_cpals(X.cuda(), dims, Ad, sweeps, 0.0, shared=shared)
    torch.cuda.synchronize()
    assert len(fits) == sweeps
    np.testing.assert_allclose(fits, fits_ref, rtol=0, atol=1e-9)
    np.testing.assert_allclose(lam.cpu().numpy(), lam_ref, rtol=1e-7)
    for m in range(len(dims)):
        got = Ad[m].cpu().numpy()
        err = np.linalg.norm(got - A_ref[m]) / np.linalg.norm(A_ref[m])
        assert err <= 1e-7, (m, err)


def test_cpals_large_rank_singular_gram_is_reported(mt):
    dims, R = (80, 75, 70), 72
    X, A0 = problem(dims, R, 36)
    Ad = [a.clone().cuda() for a in A0]
    Ad[1][:, 40] = 0.0
    before = Ad[0].clone()
    with pytest.raises(mt.MttkrpError) as e:
        mt.mttkrp_cpals(X.cuda(), dims, Ad, 2, 0.0)
    assert e.value.status == mt.MTTKRP_ERR_NUMERICAL
    torch.cuda.synchronize()
    assert torch.equal(Ad[0], before)


# Updates of several workgroups, which all read the flag that the first of them sets: a zero column in the first or the last
# place (the first pivot is bad, or only the last), 32 to 1094 tiles, ranks of every register tile, one panel and
# several above rank 64.  No factor may change.
@pytest.mark.parametrize("dims,R", [((2000, 9, 7), 8), ((70000, 6, 5), 20), ((9000, 30, 10), 64), ((70000, 9, 9), 33),
                                    ((300, 80, 75), 72), ((400, 40, 150), 130)])
@pytest.mark.parametrize("column", [0, -1])
def test_cpals_failed_update_of_several_workgroups_changes_no_factor(mt, dims, R, column):
    X, A0 = problem(dims, R, 37)
    Ad = [a.clone().cuda() for a in A0]
    Ad[1][:, column] = 0.0
    before = [a.clone() for a in Ad]
    for shared in (False, True):
        print("cp-als failed update dims=%s R=%d column=%d" % (dims, R, column), flush=True)
        with pytest.raises(mt.MttkrpError) as e:
            mt.mttkrp_cpals(X.cuda(), dims, Ad, 2, 0.0, shared=shared)
        assert e.value.status == mt.MTTKRP_ERR_NUMERICAL
        torch.cuda.synchronize()
        for a, b in zip(Ad, before):
            assert torch.equal(a, b)


def test_cpals_tolerance_stop_and_reproducibility(mt):
    from oracle import cp_als_oracle, mttkrp_oracle
    mttkrp_oracle.build()
    dims, R = (30, 24, 18), 4
    X, A0 = problem(dims, R, 21, rank_true=4, noise=0.05)
    _, _, fits_ref = cp_als_oracle.cp_als(inputs.as_ndarray_view(X, dims), [a.numpy() for a in A0], 40, 1e-4)
    Xd = X.cuda()
    runs = []
    for _ in range(2):
        Ad = [a.clone().cuda() for a in A0]
        lam, fits = mt.mttkrp_cpals(Xd, dims, Ad, 40, 1e-4)
        torch.cuda.synchronize()
        runs.append((lam.cpu().numpy().copy(), [a.cpu().numpy().copy() for a in Ad], fits))
    assert len(runs[0][2]) == len(fits_ref)                     # same stopping sweep as the oracle
    np.testing.assert_allclose(runs[0][2], fits_ref, rtol=0, atol=1e-8)
    assert runs[0][2] == runs[1][2]                             # fixed-order reductions: bit-identical reruns
    assert np.array_equal(runs[0][0], runs[1][0])
    for a, b in zip(runs[0][1], runs[1][1]):
        assert np.array_equal(a, b)


def test_cpals_recovers_an_exact_low_rank_tensor(mt):
    dims, R = (48, 40, 36), 3
    X, A0 = problem(dims, R, 31, rank_true=3)
    Xd = X.cuda()
    Ad = [a.clone().cuda() for a in A0]
    lam, fits = mt.mttkrp_cpals(Xd, dims, Ad, 300, 1e-12)
    assert fits[-1] > 1.0 - 1e-6, fits[-5:]
    assert all(b >= a - 1e-12 for a, b in zip(fits, fits[1:]))


def test_all_modes_sweep(mt, oracle):
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 1e-5)):
        dims, R = (70, 20, 9, 4), 24
        n = int(np.prod(dims))
        X = inputs.uniform(41, n, -1.0, 1.0, dtype=dtype)
        A = [inputs.uniform(42 + m, (I, R), -1.0, 1.0, dtype=dtype) for m, I in enumerate(dims)]
        Ms = mt.mttkrp_dense_all_modes(X.cuda(), dims, [a.cuda() for a in A])
        torch.cuda.synchronize()
        Xn = inputs.as_ndarray_view(X, dims)
        for k in range(len(dims)):
            ref = oracle.mttkrp(Xn, [a.numpy() for a in A], k)
            assert oracle.normwise_rel_err(Ms[k].cpu().numpy(), ref) <= tol, (dtype, k)


def test_cpals_errors(mt):
    dims = (8, 7, 6)
    X, A0 = problem(dims, 3, 51)
    Xd = X.cuda()
    with pytest.raises(mt.MttkrpError) as e:
        big = [torch.ones((I, 2049), dtype=torch.float64, device="cuda") for I in dims]
        mt.mttkrp_cpals(Xd, dims, big, 2, 0.0)
    assert e.value.status == mt.MTTKRP_ERR_UNSUPPORTED
    # a zero column makes the Gram Hadamard product singular: reported, not a crash or a NaN
    Ad = [a.clone().cuda() for a in A0]
    Ad[1][:, 2] = 0.0
    before = Ad[0].clone()
    with pytest.raises(mt.MttkrpError) as e:
        mt.mttkrp_cpals(Xd, dims, Ad, 2, 0.0)
    assert e.value.status == mt.MTTKRP_ERR_NUMERICAL
    torch.cuda.synchronize()
    assert torch.equal(Ad[0], before)                           # the failed update left A_0 as it was


# The dense steps of an update where their launches change shape: one workgroup or several (1024 rows at
# R <= 16, 512 at R <= 32; tiles of 128 and 64 rows), ranks at the register tiles' edges (16 / 17, 32 / 33, 48, 64),
# more tiles than workgroups, above rank 64 full and partial blocks of 32, factors of more than 8192 rows (four
# wavefronts a workgroup) and ranks above 1024 (the rows no longer in LDS).  Rounding differences between two
# orders of the sums grow with the condition of V (1e2 to 1e5 here) and over the sweeps: 1e-16 * 1e5 * a few
# hundred terms stays below 1e-8.
UPDATE_SHAPES = [((1024, 9, 7), 16, 2), ((1025, 9, 7), 16, 2), ((127, 129, 3), 15, 2), ((512, 20, 11), 17, 2),
                 ((513, 20, 11), 32, 2), ((65, 64, 63), 33, 2), ((130, 20, 31), 48, 2), ((9000, 30, 10), 64, 2),
                 ((70, 64, 60), 64, 2), ((8300, 30, 26), 70, 2), ((40, 39, 38), 97, 2), ((24, 23, 22, 21), 1030, 1)]


@pytest.mark.parametrize("dims,R,sweeps", UPDATE_SHAPES)
def test_cpals_update_launch_shapes(mt, dims, R, sweeps):
    from oracle import cp_als_oracle, mttkrp_oracle
    mttkrp_oracle.build()
    X, A0 = problem(dims, R, 60 + R)
    A_ref, lam_ref, fits_ref = cp_als_oracle.cp_als(inputs.as_ndarray_view(X, dims), [a.numpy() for a in A0], sweeps, 0.0)
    Ad = [a.clone().cuda() for a in A0]
    print("cp-als update dims=%s R=%d" % (dims, R), flush=True)
    lam, fits = mt.mttkrp_cpals(X.cuda(), dims, Ad, sweeps, 0.0)
    torch.cuda.synchronize()
    np.testing.assert_allclose(fits, fits_ref, rtol=0, atol=1e-8)
    np.testing.assert_allclose(lam.cpu().numpy(), lam_ref, rtol=1e-7)
    for m in range(len(dims)):
        got = Ad[m].cpu().numpy()
        err = np.linalg.norm(got - A_ref[m]) / np.linalg.norm(A_ref[m])
        assert err <= 1e-8, (m, err)


# Start factors whose Gram products lie near the ends of the exponents: pivots below 2^-1024, whose reciprocal is infinite, and
# above 2^1022, whose reciprocal is subnormal.  Values at 1e-310 carry about 45 bits, times the condition of V (11 to 450):
# below 1e-11 in a factor, 1e-9 leaves room for the second sweep.
@pytest.mark.parametrize("dims,R,low,high", [((40, 30, 20), 5, -258, 254.0), ((1100, 9, 7), 8, -258, 255.0),
                                             ((65, 64, 63), 33, -259, 253.5), ((72, 66, 70), 70, -259, 253.14)])
@pytest.mark.parametrize("end", ["low", "high"])
def test_cpals_pivots_near_the_ends_of_the_exponents(mt, dims, R, low, high, end):
    from oracle import cp_als_oracle, mttkrp_oracle
    mttkrp_oracle.build()
    X, A0 = problem(dims, R, 5)
    X = X * (2.0 ** -400 if end == "low" else 2.0 ** 300)
    A0 = [a * 2.0 ** (low if end == "low" else high) for a in A0]
    V = (A0[1].t() @ A0[1]) * (A0[2].t() @ A0[2])
    assert 1e-311 < float(V.diagonal().min()) and float(V.max()) < 1.7e308
    assert float(V.diagonal().min()) < 2.0 ** -1024 if end == "low" else float(V.diagonal().max()) > 2.0 ** 1022
    A_ref, lam_ref, fits_ref = cp_als_oracle.cp_als(inputs.as_ndarray_view(X, dims), [a.numpy() for a in A0], 2, 0.0)
    for shared in (False, True):
        Ad = [a.clone().cuda() for a in A0]
        print("cp-als exponents dims=%s R=%d %s" % (dims, R, end), flush=True)
        lam, fits = mt.mttkrp_cpals(X.cuda(), dims, Ad, 2, 0.0, shared=shared)
        np.testing.assert_allclose(fits, fits_ref, rtol=0, atol=1e-9)
        np.testing.assert_allclose(lam.cpu().numpy(), lam_ref, rtol=1e-9)
        for m in range(len(dims)):
            err = np.linalg.norm(Ad[m].cpu().numpy() - A_ref[m]) / np.linalg.norm(A_ref[m])
            assert err <= 1e-9, (m, err)


def test_cpals_norm_of_an_unaligned_tensor(mt):
    # X that starts 8 bytes off a 16-byte boundary, odd and even length: ||X|| enters every fit
    from oracle import cp_als_oracle, mttkrp_oracle
    mttkrp_oracle.build()
    for dims in ((33, 7, 5), (40, 30, 20)):
        X, A0 = problem(dims, 3, 90)
        buf = torch.zeros(X.numel() + 1, dtype=torch.float64, device="cuda")
        buf[1:] = X.cuda()
        Ad = [a.clone().cuda() for a in A0]
        _, _, fits_ref = cp_als_oracle.cp_als(inputs.as_ndarray_view(X, dims), [a.numpy() for a in A0], 2, 0.0)
        _, fits = mt.mttkrp_cpals(buf[1:], dims, Ad, 2, 0.0)
        np.testing.assert_allclose(fits, fits_ref, rtol=0, atol=1e-10)
