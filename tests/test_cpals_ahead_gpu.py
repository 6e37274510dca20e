"""CP-ALS enqueues sweeps ahead of the records that end the iteration: it still stops after the sweep in which the fit settles,
with the factors, weights and fits of that sweep, runs past the number of records that one read holds, and enqueues no
more behind its last sweep than the waits that this saves are worth.  The MTTKRPs that it enqueues are counted."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

RECORDS = 16        # sweeps between two reads at most
WAIT_US = 40.0      # what a read costs
AHEAD_US = 2000.0   # work ahead of a read


def problem(dims, rank, seed, noise):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    U = [torch.randn(I, rank, dtype=torch.float64, device="cuda", generator=gen) for I in dims]
    low = (U[1][:, None, :] * U[0][None, :, :]).reshape(-1, rank)            # first index fastest
    X = (U[2] @ low.t()).reshape(-1)
    X += noise * torch.randn(X.shape, dtype=torch.float64, device="cuda", generator=gen)
    return X, [torch.rand(I, rank, dtype=torch.float64, device="cuda", generator=gen) for I in dims]


def run(mt, X, dims, A0, iters, tol, shared=False):
    """Factors, weights, fits, sweeps enqueued (separate passes only) and microseconds for each of them."""
    A = [a.clone() for a in A0]
    torch.cuda.synchronize()
    mt.mttkrp_timing_enable(True)
    t0 = time.perf_counter()
    try:
        lam, fits = mt.mttkrp_cpals(X, dims, A, iters, tol, shared=shared)
        torch.cuda.synchronize()
        took = 1e6 * (time.perf_counter() - t0)
        enqueued = mt.mttkrp_timing_count() / len(dims)
    finally:
        mt.mttkrp_timing_enable(False)
    return [a.cpu().numpy() for a in A], lam.cpu().numpy(), list(fits), enqueued, took / max(enqueued, 1)


def same(a, b):
    assert a[2] == b[2]
    np.testing.assert_array_equal(a[1], b[1])
    for x, y in zip(a[0], b[0]):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("dims,rank,shared,tol", [((30, 20, 25), 4, False, 1e-5), ((30, 20, 25), 4, True, 1e-5),
                                                  ((24, 22, 21), 70, False, 2e-3), ((170, 160, 170), 3, False, 1e-5)])
def test_stops_with_the_state_of_the_last_sweep(dims, rank, shared, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    X, A0 = problem(dims, rank, 7, 0.05)
    print("cp-als ahead dims=%s R=%d shared=%s" % (dims, rank, shared), flush=True)
    a = run(mt, X, dims, A0, 90, tol, shared)
    n = len(a[2])
    assert 2 < n < 90, n
    changes = np.abs(np.diff(a[2]))
    assert changes[-1] < tol and (changes[:-1] >= tol).all()
    same(a, run(mt, X, dims, A0, n, 0.0, shared))


def test_stops_inside_a_group_of_sweeps():
    """Tolerances just above each of a run's changes, so that it stops at every sweep, in the middle of groups too: then
    sweeps are enqueued behind the last one, and leave everything as it is."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    dims, rank = (30, 20, 25), 5
    inside = 0
    for seed in range(4):
        X, A0 = problem(dims, rank, seed, 0.3)
        changes = np.abs(np.diff(run(mt, X, dims, A0, 60, 0.0)[2]))
        for n in range(4, 60, 2):
            tol = 1.001 * changes[n - 2]
            if tol == 0.0:               # (runs all sweeps)
                continue
            a = run(mt, X, dims, A0, 60, tol)
            m = len(a[2])
            print("cp-als inside seed=%d n=%d sweeps=%d enqueued=%g" % (seed, n, m, a[3]), flush=True)
            assert m <= n
            if a[3] > m:
                inside += 1
                same(a, run(mt, X, dims, A0, m, 0.0))
    assert inside >= 1


@pytest.mark.parametrize("dims,rank", [((30, 20, 25), 4), ((150, 160, 140), 8), ((330, 320, 300), 6), ((450, 430, 440), 6)])
def test_sweeps_behind_the_last_one_cost_less_than_the_waits_saved(dims, rank):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    for seed, noise, tol in ((1, 1.0, 1e-4), (2, 3.0, 1e-4), (3, 0.1, 1e-4), (1, 1.0, 1e-6), (2, 3.0, 1e-6), (3, 0.1, 1e-6)):
        X, A0 = problem(dims, rank, seed, noise)
        us = min(run(mt, X, dims, A0, 12, 0.0)[4] for _ in range(3))
        a = run(mt, X, dims, A0, 100, tol)
        n, wasted = len(a[2]), a[3] - len(a[2])
        print("cp-als waste dims=%s seed=%d tol=%g sweeps=%d wasted=%g of %.0f us" % (dims, seed, tol, n, wasted, us), flush=True)
        # (twice that: this sweep time has the set-up and the timing's events in it, the driver's own is the fastest group's)
        assert wasted * us <= 2.0 * WAIT_US * n


@pytest.mark.parametrize("dims,rank", [((100, 80, 60), 10), ((60, 60, 60), 200), ((40, 45, 50), 600)])
def test_a_failure_is_reported_after_the_work_ahead(dims, rank):
    """A factor with a zero column: V is singular in the first update, and what was enqueued behind it is what goes ahead."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    X, A0 = problem(dims, rank, 5, 0.1)
    us = min(run(mt, X, dims, A0, 4, 0.0)[4] for _ in range(3))
    bad = [a.clone() for a in A0]
    bad[1][:, rank // 2] = 0.0
    mt.mttkrp_timing_enable(True)
    try:
        with pytest.raises(mt.MttkrpError):
            mt.mttkrp_cpals(X, dims, bad, 40, 0.0)
        enqueued = mt.mttkrp_timing_count() / len(dims)
    finally:
        mt.mttkrp_timing_enable(False)
    print("cp-als failure dims=%s R=%d: %g sweeps of %.0f us ahead" % (dims, rank, enqueued, us), flush=True)
    assert 1 <= enqueued <= max(1, min(RECORDS, 2 * AHEAD_US / us))       # (an estimate: within a factor of two)


def test_more_sweeps_than_one_read_holds():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    dims = (12, 11, 10)
    X, A0 = problem(dims, 1, 8, 0.1)         # (rank one: no swamps, every sweep is as good as its start)
    a = run(mt, X, dims, A0, 131, 0.0)
    assert len(a[2]) == 131 and all(np.isfinite(a[2])) and max(np.abs(np.diff(a[2][-20:]))) < 1e-9
    b = run(mt, X, dims, A0, 60, 0.0)
    c = run(mt, X, dims, [torch.from_numpy(x).cuda() for x in b[0]], 71, 0.0)
    # (lambda is not an input: a sweep starts from the factors alone)
    np.testing.assert_allclose(b[2] + c[2], a[2], rtol=0, atol=1e-12)
