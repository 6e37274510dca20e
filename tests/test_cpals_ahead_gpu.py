"""CP-ALS enqueues sweeps ahead of the records that end the iteration: it still stops after the sweep in which the fit settles,
with the factors, weights and fits of that sweep, and runs past the number of records that one read holds."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def problem(dims, rank, seed, noise):
    rng = np.random.default_rng(seed)
    U = [rng.standard_normal((I, rank)) for I in dims]
    X = np.einsum("ar,br,cr->abc", *U)
    X = X + noise * rng.standard_normal(dims)
    return torch.from_numpy(np.ascontiguousarray(X.reshape(-1, order="F"))).cuda(), [rng.uniform(0.0, 1.0, (I, rank)) for I in dims]


def run(mt, X, dims, A0, iters, tol, shared):
    A = [torch.from_numpy(a).cuda() for a in A0]
    lam, fits = mt.mttkrp_cpals(X, dims, A, iters, tol, shared=shared)
    torch.cuda.synchronize()
    return [a.cpu().numpy() for a in A], lam.cpu().numpy(), list(fits)


@pytest.mark.parametrize("dims,rank,shared,tol", [((30, 20, 25), 4, False, 1e-5), ((30, 20, 25), 4, True, 1e-5),
                                                  ((24, 22, 21), 70, False, 2e-3), ((170, 160, 170), 3, False, 1e-5)])
def test_stops_with_the_state_of_the_last_sweep(dims, rank, shared, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    X, A0 = problem(dims, rank, 7, 0.05)
    print("cp-als ahead dims=%s R=%d shared=%s" % (dims, rank, shared), flush=True)
    A, lam, fits = run(mt, X, dims, A0, 90, tol, shared)
    n = len(fits)
    assert 2 < n < 90, n
    changes = np.abs(np.diff(fits))
    assert changes[-1] < tol and (changes[:-1] >= tol).all()
    B, lam_b, fits_b = run(mt, X, dims, A0, n, 0.0, shared)
    assert fits == fits_b
    np.testing.assert_array_equal(lam, lam_b)
    for a, b in zip(A, B):
        np.testing.assert_array_equal(a, b)


def test_more_sweeps_than_one_read_holds():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    dims = (12, 11, 10)
    X, A0 = problem(dims, 1, 8, 0.1)         # (rank one: no swamps, every sweep is as good as its start)
    A, _, fits = run(mt, X, dims, A0, 131, 0.0, False)
    assert len(fits) == 131 and all(np.isfinite(fits)) and max(np.abs(np.diff(fits[-20:]))) < 1e-9
    B, _, fits_b = run(mt, X, dims, A0, 60, 0.0, False)
    C, _, fits_c = run(mt, X, dims, B, 71, 0.0, False)
    # (lambda is not an input: a sweep starts from the factors alone)
    np.testing.assert_allclose(fits_b + fits_c, fits, rtol=0, atol=1e-12)
