"""The sum of the partial slots by one thread an entry: few slots (1 to 4, 5 to 16) and large outputs with more of them, with and without
weights and accumulation, against a float64 product with the explicit Khatri-Rao matrix.  Tolerance: sums of n products of random
sign in any order, 8 u sqrt(n) of their norm, and one rounding to the data type."""
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")

CASES = [((33, 500, 64), 17, 1, "f64", 1, 4), ((1000, 300, 40), 50, 1, "f64", 1, 16), ((16641, 60, 40), 10, 0, "f64", 5, 16),
         ((33, 4000, 64), 40, 1, "f32", 1, 16), ((13200, 100, 40), 10, 0, "f32", 17, 255), ((3400, 300, 50), 40, 0, "f32", 17, 255)]


@pytest.mark.gpu
@pytest.mark.parametrize("dims,R,k,dtype,low,high", CASES)
def test_few_slots_and_large_outputs(dims, R, k, dtype, low, high):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_14891_amd import binding as mt
    T = torch.float64 if dtype == "f64" else torch.float32
    slots = int(re.findall(r"slots=(\d+)", mt.mttkrp_plan_describe(dims, R, k, T.itemsize))[-1])
    assert low <= slots <= high
    print("combine dims=%s R=%d k=%d %s slots=%d" % (dims, R, k, dtype, slots), flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(R)
    X = torch.randn(int(np.prod(dims)), dtype=T, device="cuda", generator=gen)
    A = [torch.randn((n, R), dtype=T, device="cuda", generator=gen) for n in dims]
    lam = torch.rand(R, dtype=T, device="cuda", generator=gen) + 0.5
    M0 = torch.randn((dims[k], R), dtype=T, device="cuda", generator=gen)
    rest = [m for m in range(3) if m != k]
    krp = (A[rest[1]].double()[:, None, :] * A[rest[0]].double()[None, :, :]).reshape(-1, R)
    Xk = X.double().view(dims[2], dims[1], dims[0]).permute(2, 1, 0).permute(k, rest[1], rest[0]).reshape(dims[k], -1)
    want = Xk @ krp
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    bound = 8.0 * u * np.sqrt(krp.shape[0])
    got = mt.mttkrp_dense(X, dims, A, k)
    assert float((got.double() - want).norm() / want.norm()) <= bound
    acc = mt.mttkrp_dense(X, dims, A, k, M=M0.clone(), lam=lam, beta=0.5)
    want = want * lam.double() + 0.5 * M0.double()
    assert float((acc.double() - want).norm() / want.norm()) <= bound
