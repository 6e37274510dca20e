"""The CP-ALS benchmark's MTTKRP time: calls of discarded sweeps apart, calls whose events are no longer kept scaled in."""
import pytest

from paper_2510_14891_amd import cpals_bench


@pytest.mark.parametrize("ndim,sweeps,discarded", [(5, 12, 0), (3, 14, 4), (3, 200, 0), (5, 150, 3), (8, 64, 15)])
def test_mttkrp_times(ndim, sweeps, discarded):
    asked = []

    def get(i):
        assert n - cpals_bench.KEPT_CALLS <= i < n
        asked.append(i)
        return (2.0 + i % ndim, 0.5) if i < ndim * sweeps else (100.0, 1.0)

    n = ndim * (sweeps + discarded)
    wanted, rest = cpals_bench.mttkrp_times(get, n, ndim * sweeps)
    per_sweep = sum(2.5 + m for m in range(ndim))
    # (the kept calls need not begin with a sweep: within one sweep's spread of their mean)
    assert wanted == pytest.approx(sweeps * per_sweep, rel=0.0 if n <= cpals_bench.KEPT_CALLS else ndim * ndim / cpals_bench.KEPT_CALLS, abs=1e-9)
    assert rest == pytest.approx(101.0 * ndim * discarded)
    assert len(asked) == min(n, cpals_bench.KEPT_CALLS)
