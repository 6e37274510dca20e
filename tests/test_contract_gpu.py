"""The contraction over the leading index through LDS (contract.hip) and the mode results taken from it, against the CPU
oracle at the edges of its tiles: stages of 32 (fp64) and 64 (fp32) rows, tiles of 64 and 128 columns, 16- to 64-column
outputs, row splits, leading dimensions, tensors that begin 8 (4) bytes off a line, non-finite values beside the masked
rows.  Tolerances as everywhere: 1e-12 and 1e-5, normwise."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_14891_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-12, torch.float32: 1e-5}


@pytest.fixture(scope="module")
def mt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding
    binding.lib()
    yield binding
    for key in ("lds_contract", "target_items", "max_steps"):
        binding.mttkrp_tune_set(key, 0)


# (P, Q, R): first and last stage whole, one row, one row short; one column, tiles less one, whole, plus one
EDGES = [(384, 1, 2), (385, 63, 16), (415, 64, 17), (416, 65, 31), (447, 127, 32), (448, 128, 4), (513, 129, 33),
         (1001, 200, 48), (2049, 257, 20), (640, 300, 5), (401, 900, 10), (5000, 70, 7)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
# ("lds_contract" = 1: also where the tiles of this kernel hold many more columns than the other's)
@pytest.mark.parametrize("tune", [{}, {"target_items": 9}, {"max_steps": 8}, {"lds_contract": 1},
                                  {"lds_contract": 1, "target_items": 9}, {"lds_contract": 1, "max_steps": 8}])
@pytest.mark.parametrize("P,Q,R", EDGES)
def test_contraction_through_lds(mt, oracle, P, Q, R, tune, dtype):
    if dtype == torch.float32:
        R = max(4, R + (16 if R == 48 else 0))         # up to 64 output columns in fp32
    buf = inputs.uniform(5, P * Q + 1, -1.0, 1.0, dtype=dtype)
    wide = inputs.uniform(6, (P, R + 3), -1.0, 1.0, dtype=dtype)
    K = wide[:, :R].contiguous()
    for off in (0, 1):                                   # lines and columns aligned or not
        X = buf[off:off + P * Q].contiguous()
        ref = oracle.mttkrp(inputs.as_ndarray_view(X, (P, Q)), [K.numpy(), np.zeros((Q, R), dtype=K.numpy().dtype)], 1)
        Xd = buf.cuda()[off:off + P * Q]
        for key, val in tune.items():
            mt.mttkrp_tune_set(key, val)
        print("contract P=%d Q=%d R=%d %s off=%d" % (P, Q, R, tune, off), flush=True)
        T = torch.full((Q, R + 2), 3.0, dtype=dtype, device="cuda")
        mt.mttkrp_contract_leading(Xd, P, Q, wide.cuda()[:, :R], T_out=T[:, :R])
        again = mt.mttkrp_contract_leading(Xd, P, Q, K.cuda())
        for key in tune:
            mt.mttkrp_tune_set(key, 0)
        assert oracle.normwise_rel_err(T[:, :R].cpu().numpy(), ref) <= TOL[dtype]
        assert torch.equal(T[:, :R], again) and bool((T[:, R:] == 3.0).all())


# Modes that run on the contraction and the weighted sum of its result (asserted from the plan, with the key that leaves
# only the limits on sizes): one and several segments of that sum, one and several row splits, one to three
# blocks of output columns, modes of one entry, the output mode first, between and last among the others.
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dims,R", [((3000, 20, 20), 32), ((2573, 7, 9), 5), ((4001, 3, 1, 2, 4), 17), ((9000, 65, 3), 16),
                                    ((4000, 30, 29), 8), ((30000, 3, 5), 4), ((840, 2, 3, 2, 1), 4), ((12024, 28, 1), 5),
                                    ((2601, 3, 301), 48), ((500, 2, 5, 2), 20)])
def test_modes_from_the_contraction(mt, oracle, dims, R, dtype):
    X = inputs.uniform(7, int(np.prod(dims)), -1.0, 1.0, dtype=dtype)
    A = [inputs.uniform(8 + m, (I, R), -1.0, 1.0, dtype=dtype) for m, I in enumerate(dims)]
    Xn, An = inputs.as_ndarray_view(X, dims), [a.numpy() for a in A]
    Xd, Ad = X.cuda(), [a.cuda() for a in A]
    lam = inputs.uniform(9, R, 0.5, 1.5, dtype=dtype)
    for k in range(1, len(dims)):
        mt.mttkrp_tune_set("small_route", 2)
        mt.mttkrp_tune_set("lds_contract", 1)
        plan = mt.mttkrp_plan_describe(dims, R, k, X.element_size())
        print("modes from the contraction dims=%s R=%d k=%d %s" % (dims, R, k, plan), flush=True)
        assert "lds=1" in plan or (dims, k) in [((9000, 65, 3), 2), ((2601, 3, 301), 1)]       # (streaming plans)
        ref = oracle.mttkrp(Xn, An, k)
        got = mt.mttkrp_dense(Xd, dims, Ad, k)
        wide = [torch.full((I, R + 1), float("nan"), dtype=dtype, device="cuda") for I in dims]
        for w, a in zip(wide, Ad):
            w[:, :R] = a
        Mw = torch.full((dims[k], R + 3), 1.0, dtype=dtype, device="cuda")
        mt.mttkrp_dense_ld(Xd, dims, [w[:, :R] for w in wide], k, Mw[:, :R], R, lam=lam.cuda(), beta=0.5)
        mt.mttkrp_tune_set("small_route", 0)
        mt.mttkrp_tune_set("lds_contract", 0)
        assert oracle.normwise_rel_err(got.cpu().numpy(), ref) <= TOL[dtype], k
        ref2 = oracle.mttkrp(Xn, An, k, lam=lam.numpy()) + 0.5
        assert oracle.normwise_rel_err(Mw[:, :R].cpu().numpy(), ref2) <= TOL[dtype], k
        assert bool((Mw[:, R:] == 1.0).all())


# Ranks below a thread's four consecutive columns, and ranks whose last group of four overlaps the one before it.
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("R", [2, 3, 6, 7, 9, 18, 30, 31])
def test_modes_from_the_contraction_at_ragged_ranks(mt, oracle, R, dtype):
    dims = (3000, 20, 21)
    X = inputs.uniform(17, int(np.prod(dims)), -1.0, 1.0, dtype=dtype)
    A = [inputs.uniform(18 + m, (I, R), -1.0, 1.0, dtype=dtype) for m, I in enumerate(dims)]
    Xn, An = inputs.as_ndarray_view(X, dims), [a.numpy() for a in A]
    Xd, Ad = X.cuda(), [a.cuda() for a in A]
    for k in (1, 2):
        mt.mttkrp_tune_set("small_route", 2)
        mt.mttkrp_tune_set("lds_contract", 1)
        plan = mt.mttkrp_plan_describe(dims, R, k, X.element_size())
        print("modes from the contraction, ragged rank dims=%s R=%d k=%d %s" % (dims, R, k, plan), flush=True)
        M = torch.full((dims[k], R + 3), 1.0, dtype=dtype, device="cuda")
        mt.mttkrp_dense_ld(Xd, dims, Ad, k, M[:, :R], R)
        mt.mttkrp_tune_set("small_route", 0)
        mt.mttkrp_tune_set("lds_contract", 0)
        assert "lds=1" in plan or (R < 4 and dtype == torch.float32)          # (streaming plans)
        assert oracle.normwise_rel_err(M[:, :R].cpu().numpy(), oracle.mttkrp(Xn, An, k)) <= TOL[dtype], k
        assert bool((M[:, R:] == 1.0).all())


# The same with two and three blocks of output columns, which this route takes for longer first modes only: against float64
# products on the GPU.
@pytest.mark.parametrize("dims,R,k,dtype", [((120000, 3, 130), 20, 2, torch.float64), ((120000, 3, 130), 20, 2, torch.float32),
                                            ((100001, 20, 20), 17, 1, torch.float64), ((280001, 20, 20), 48, 2, torch.float64),
                                            ((1100000, 20, 20), 32, 1, torch.float32)])
def test_modes_from_the_contraction_at_higher_ranks(mt, dims, R, k, dtype):
    plan = mt.mttkrp_plan_describe(dims, R, k, torch.empty((), dtype=dtype).element_size())
    print("modes from the contraction dims=%s R=%d k=%d %s" % (dims, R, k, plan), flush=True)
    assert "shape=rows" in plan and "lds=1" in plan
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    X = torch.rand((dims[2], dims[1], dims[0]), dtype=dtype, device="cuda", generator=g) - 0.5
    A = [torch.rand((I, R), dtype=dtype, device="cuda", generator=g) - 0.5 for I in dims]
    S = torch.stack([X[i].double() @ A[0].double() for i in range(dims[2])])          # i_2, i_1, j
    want = torch.zeros((dims[k], R), dtype=torch.float64, device="cuda")
    for i in range(dims[3 - k]):
        want += (S[i] if k == 1 else S[:, i]) * A[3 - k][i].double()
    got = mt.mttkrp_dense(X.view(-1), dims, A, k)
    assert float((got.double() - want).norm() / want.norm()) <= TOL[dtype]
    lam = torch.rand(R, dtype=dtype, device="cuda", generator=g) + 0.5
    acc = mt.mttkrp_dense(X.view(-1), dims, A, k, M=got.clone(), lam=lam, beta=-0.5)
    want = want * lam.double() - 0.5 * got.double()
    assert float((acc.double() - want).norm() / want.norm()) <= 2.0 * TOL[dtype]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_contraction_non_finite_rows_beside_masked_ones(mt, dtype):
    # the last stage repeats rows of the one before and masks them: an infinity there must enter once and not as inf * 0
    P, Q, R = 401, 70, 6
    X = torch.ones((Q, P), dtype=dtype, device="cuda")
    K = torch.ones((P, R), dtype=dtype, device="cuda")
    X[3, 380] = float("inf")
    K[390, 2] = float("inf")
    T = mt.mttkrp_contract_leading(X.view(-1), P, Q, K)
    want = torch.full((Q, R), float(P), dtype=dtype, device="cuda")
    want[3, :] = float("inf")
    want[:, 2] = float("inf")
    assert torch.equal(T, want)


# Calls whose row splits in this kernel are longer than the chains of the kernel that "lds_contract" = 2 selects: both add the same number
# of products in single precision and the rest in double precision, so their errors agree up to the scatter of
# tens of thousands of outputs (1.25) and the rounding of a result (2e-8).  One to four blocks of output columns, tiles of 64 and
# 128 columns, splits of whole stages and not.
@pytest.mark.parametrize("P,Q,R", [(3978, 2857, 17), (4096, 2000, 32), (5000, 9000, 10), (16641, 500, 4), (20000, 130, 10),
                                   (8000, 3000, 40), (8000, 3000, 64), (30000, 130, 20), (300000, 300, 32), (1300, 20000, 24)])
def test_single_precision_chains_are_no_longer_than_the_other_kernels(mt, P, Q, R):
    g = torch.Generator(device="cuda")
    g.manual_seed(P)
    for signed in (False, True):
        X = torch.rand((Q, P), dtype=torch.float32, device="cuda", generator=g) - 0.5 * signed
        K = torch.rand((P, R), dtype=torch.float32, device="cuda", generator=g) - 0.5 * signed
        W = torch.cat([X[q:q + 512].double() @ K.double() for q in range(0, Q, 512)])
        err = []
        for v in (1, 2):
            mt.mttkrp_tune_set("lds_contract", v)
            print("contract chains P=%d Q=%d R=%d lds_contract=%d" % (P, Q, R, v), flush=True)
            T = mt.mttkrp_contract_leading(X.view(-1), P, Q, K)
            mt.mttkrp_tune_set("lds_contract", 0)
            err.append(float((T.double() - W).norm() / W.norm()))
        assert err[0] <= 1.25 * err[1] + 2e-8, err
