"""The one-launch path for small tensors (small.hip) against the CPU oracle: sizes at the edges of its tiles (16-row
blocks, batches of 16 and 32 columns, 16 wavefronts, 16- to 64-column chunks of the output), extents of one, two to
eight modes, one workgroup per output row and several with a combine launch, weights and accumulation, leading
dimensions, non-finite values.  Tolerances are those of every parity test: 1e-12 (fp64) and 1e-5 (fp32), normwise."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_14891_amd import inputs

TOL = {torch.float64: 1e-12, torch.float32: 1e-5}

SHAPES = [((64, 64, 64), 16), ((1, 1), 1), ((16, 32), 2), ((17, 33), 15), ((15, 129), 17), ((33, 31, 5), 32),
          ((64, 1, 65), 33), ((1, 70, 9), 48), ((31, 2, 1, 40), 49), ((3, 1, 1, 7), 64), ((48, 16, 3, 2), 65),
          ((9, 8, 7, 3, 2), 100), ((5, 4, 3, 2, 2, 3), 3), ((2, 3, 2, 2, 3, 2, 2, 3), 20), ((130, 4, 31), 130),
          ((300, 5, 3), 7), ((7, 300, 2), 9)]


@pytest.fixture(scope="module")
def mt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding
    binding.lib()
    yield binding
    binding.mttkrp_tune_set("small_route", 0)
    binding.mttkrp_tune_set("small_groups", 0)


def make(dims, R, dtype, seed):
    X = inputs.uniform(seed, int(np.prod(dims)), -1.0, 1.0, dtype=dtype)
    A = [inputs.uniform(seed + 100 + m, (I, R), -1.0, 1.0, dtype=dtype) for m, I in enumerate(dims)]
    return X, A


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("groups", [1, 4])
@pytest.mark.parametrize("dims,R", SHAPES)
def test_small_route_matches_the_oracle(mt, oracle, dims, R, groups, dtype):
    X, A = make(dims, R, dtype, 11)
    Xd, Ad = X.cuda(), [a.cuda() for a in A]
    An, Xn = [a.numpy() for a in A], inputs.as_ndarray_view(X, dims)
    lam = inputs.uniform(12, R, 0.5, 2.0, dtype=dtype)
    mt.mttkrp_tune_set("small_route", 1)
    mt.mttkrp_tune_set("small_groups", groups)
    for k in range(len(dims)):
        assert "small_route=1" in mt.mttkrp_plan_describe(dims, R, k, X.element_size())
        print("small route dims=%s R=%d k=%d groups=%d" % (dims, R, k, groups), flush=True)
        ref = oracle.mttkrp(Xn, An, k)
        f = list(Ad)
        f[k] = None
        got = mt.mttkrp_dense(Xd, dims, f, k)
        assert oracle.normwise_rel_err(got.cpu().numpy(), ref) <= TOL[dtype]
        assert torch.equal(got, mt.mttkrp_dense(Xd, dims, f, k))        # fixed order
        M = inputs.uniform(13 + k, (dims[k], R), -1.0, 1.0, dtype=dtype)
        want = 0.5 * M.numpy().astype(np.float64) + ref * lam.numpy()
        acc = mt.mttkrp_dense(Xd, dims, f, k, M=M.cuda(), lam=lam.cuda(), beta=0.5)
        scale = np.linalg.norm(want) / max(np.linalg.norm(ref), 1e-300)
        assert oracle.normwise_rel_err(acc.cpu().numpy(), want) <= TOL[dtype] * max(1.0, 1.0 / scale)
        # blocks of wider arrays
        wide = [torch.zeros((I, R + 3), dtype=dtype, device="cuda") for I in dims]
        for w, a in zip(wide, Ad):
            w[:, :R] = a
        Mw = torch.full((dims[k], R + 5), 7.0, dtype=dtype, device="cuda")
        mt.mttkrp_dense_ld(Xd, dims, wide, k, Mw, R)
        assert torch.equal(Mw[:, :R], got) and bool((Mw[:, R:] == 7.0).all())
    mt.mttkrp_tune_set("small_route", 0)
    mt.mttkrp_tune_set("small_groups", 0)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_small_route_non_finite_values(mt, oracle, dtype):
    for dims, R in (((40, 7, 5), 6), ((70, 9, 3, 2), 20), ((33, 5), 3)):
        X, A = make(dims, R, dtype, 21)
        X, A = X.abs() + 0.1, [a.abs() + 0.1 for a in A]
        inputs.as_ndarray_view(X, dims)[(dims[0] - 1, dims[1] - 1) + (0,) * (len(dims) - 2)] = np.inf
        A[1][dims[1] - 1, R - 1] = np.inf
        for k in range(len(dims)):
            ref = oracle.mttkrp(inputs.as_ndarray_view(X, dims), [a.numpy() for a in A], k)
            for groups in (1, 4):
                mt.mttkrp_tune_set("small_route", 1)
                mt.mttkrp_tune_set("small_groups", groups)
                got = mt.mttkrp_dense(X.cuda(), dims, [a.cuda() for a in A], k).cpu().numpy()
                mt.mttkrp_tune_set("small_route", 0)
                mt.mttkrp_tune_set("small_groups", 0)
                assert np.array_equal(np.isinf(got), np.isinf(ref)) and not np.isnan(got).any(), (dims, k)
                fin = np.isfinite(ref)
                assert oracle.normwise_rel_err(np.where(fin, got, 0.0), np.where(fin, ref, 0.0)) <= TOL[dtype]


@pytest.mark.gpu
def test_factors_inside_arrays_beyond_32_bit_offsets(mt, oracle):
    """34 rows that lie 2^27 - 1 values apart (18 GB of single precision): a row offset formed in 32 bits wraps and reads
    another place of the same array."""
    dims, R, ld = (34, 34, 34), 16, 2 ** 27 - 1
    X, A = make(dims, R, torch.float32, 61)
    big = torch.full((34 * ld,), float("nan"), dtype=torch.float32, device="cuda")
    wide = [big.as_strided((34, R), (ld, 1), 64 * m) for m in range(2)] + [A[2].cuda()]
    for w, a in zip(wide, A[:2]):
        w.copy_(a)
    lam = inputs.uniform(62, R, 0.5, 2.0, dtype=torch.float32)
    for k in range(3):
        assert "small_route=1" in mt.mttkrp_plan_describe(dims, R, k, 4)
        ref = oracle.mttkrp(inputs.as_ndarray_view(X, dims), [a.numpy() for a in A], k)
        print("wide leading dimensions k=%d" % k, flush=True)
        M = torch.full((dims[k], R), 1.0, dtype=torch.float32, device="cuda")
        mt.mttkrp_dense_ld(X.cuda(), dims, wide, k, M, R)
        assert oracle.normwise_rel_err(M.cpu().numpy(), ref) <= TOL[torch.float32], k
        M = torch.full((dims[k], R), 1.0, dtype=torch.float32, device="cuda")
        mt.mttkrp_dense_ld(X.cuda(), dims, wide, k, M, R, lam=lam.cuda(), beta=0.5)
        want = ref * lam.numpy() + 0.5
        assert oracle.normwise_rel_err(M.cpu().numpy(), want) <= TOL[torch.float32], k


def test_small_route_is_for_small_tensors():
    from paper_2510_14891_amd import binding
    for dims, R, k, sb in (((64, 64, 64), 16, 0, 8), ((100, 80, 60), 10, 1, 8), ((20, 10, 5), 4, 2, 4)):
        assert "small_route=1" in binding.mttkrp_plan_describe(dims, R, k, sb)
    for dims, R, k, sb in (((1024, 1024, 512), 32, 0, 8), ((129, 129, 129, 12, 39), 10, 3, 8), ((48,) * 5, 64, 1, 4),
                           ((300, 300, 300), 16, 1, 8)):
        assert "small_route=1" not in binding.mttkrp_plan_describe(dims, R, k, sb)
    # a decomposition that a caller asks for is the one that runs
    binding.mttkrp_tune_set("row_blocks", 2)
    try:
        assert "small_route=1" not in binding.mttkrp_plan_describe((64, 64, 64), 16, 1, 8)
    finally:
        binding.mttkrp_tune_set("row_blocks", 0)


# Calls that took the kernel for small tensors and were 1.3 to 2.1 times slower there than without it: large ones, high ranks
# beside few or many columns, two modes.
@pytest.mark.parametrize("b,dims,R,k", [(8, (4558, 14055), 4, 0), (8, (93, 132680), 5, 1), (8, (119, 248464), 4, 0),
                                        (8, (9, 76, 72, 4, 7), 61, 1), (8, (24, 66, 20, 31), 122, 1), (8, (16, 3, 95, 318), 53, 2),
                                        (8, (11, 9, 10, 7, 15, 10), 47, 5), (8, (1293, 14063), 6, 0), (8, (141, 413, 41), 51, 2)])
def test_calls_that_the_small_kernel_slows_down_do_without_it(b, dims, R, k):
    from paper_2510_14891_amd import binding
    assert "small_route=1" not in binding.mttkrp_plan_describe(dims, R, k, b)


@pytest.mark.gpu
def test_workspace_hand_over_and_growth_without_events(mt, oracle):
    """No event follows a call until a ninth stream takes over a workspace: growth on a stream with a call in
    flight, then nine streams, then growth again; every result against the oracle."""
    mt.mttkrp_release()
    mt.mttkrp_tune_set("small_route", 2)
    probs = []
    for i in range(10):
        dims, R = (48 + 16 * i, 90 + 7 * i, 60 + 3 * i), 16
        X, A = make(dims, R, torch.float64, 300 + i)
        ref = oracle.mttkrp(inputs.as_ndarray_view(X, dims), [a.numpy() for a in A], 0)
        probs.append((dims, X.cuda(), [a.cuda() for a in A], ref))
    s0 = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s0):
        outs = [mt.mttkrp_dense(X, dims, A, 0) for dims, X, A, _ in probs]      # grows several times on one stream
    streams = [torch.cuda.Stream() for _ in range(10)]
    for _ in range(2):
        for s, (dims, X, A, _) in zip(streams, probs):
            with torch.cuda.stream(s):
                outs.append(mt.mttkrp_dense(X, dims, A, 0))
    torch.cuda.synchronize()
    mt.mttkrp_tune_set("small_route", 0)
    for i, M in enumerate(outs):
        assert oracle.normwise_rel_err(M.cpu().numpy(), probs[i % 10][3]) <= 1e-12, i


# The decompositions that the parity tests look for at default settings, on shapes that the small kernel now takes:
# the same tests with that kernel switched off.
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", ["test_fused_row_modes", "test_paired_rows_for_the_first_two_modes",
                                  "test_non_finite_values_propagate_as_in_the_definition", "test_ex_lambda_and_beta"])
def test_general_route_on_small_shapes(mt, oracle, name, dtype):
    import test_parity_gpu as parity
    mt.mttkrp_tune_set("small_route", 2)
    try:
        args = {"mt": mt, "oracle": oracle, "dtype": dtype}
        getattr(parity, name)(**args)
    finally:
        mt.mttkrp_tune_set("small_route", 0)


@pytest.mark.gpu
def test_general_route_on_the_small_shape_list(mt, oracle):
    import test_parity_gpu as parity
    mt.mttkrp_tune_set("small_route", 2)
    try:
        for dims, R in parity.SMALL:
            for dtype in (torch.float64, torch.float32):
                parity.check_all_modes(mt, oracle, dims, R, dtype, seed=7)
    finally:
        mt.mttkrp_tune_set("small_route", 0)
