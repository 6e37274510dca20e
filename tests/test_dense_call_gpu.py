"""mttkrp_dense() with and without the extension module: the same results bit for bit, the same refusals in the same words, for every form
of argument that the Python code takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


def outcome(mt, native, args, kw):
    mt._dense_call = None if native else (lambda *a: None)
    try:
        M = mt.mttkrp_dense(*args, **kw)
        torch.cuda.synchronize()
        return "ok", M.clone(), (kw.get("M") is M) if kw.get("M") is not None else None
    except (ValueError, TypeError, IndexError, AttributeError, mt.MttkrpError) as e:
        return type(e).__name__, str(e), None
    finally:
        mt._dense_call = None


class Sub(torch.Tensor):
    pass


def forms(T):
    dims, R = (6, 5, 4), 3
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    X = torch.randn(120, dtype=T, device="cuda", generator=g)
    A = [torch.randn((n, R), dtype=T, device="cuda", generator=g) for n in dims]
    M = torch.randn((5, R), dtype=T, device="cuda", generator=g)
    lam = torch.rand(R, dtype=T, device="cuda", generator=g)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    other = torch.float32 if T is torch.float64 else torch.float64
    wide = torch.randn((5, 2 * R), dtype=T, device="cuda", generator=g)
    yield "plain", (X, dims, A, 1), {}
    yield "lists", (X, list(dims), tuple(A), 1), {}
    yield "size", (X, torch.Size(dims), A, 1), {}
    yield "shaped X", (X.view(4, 5, 6), dims, A, 1), {}
    yield "numpy extents", (X, np.array(dims), A, np.int64(1)), {}
    yield "no A_k", (X, dims, [A[0], None, A[2]], 1), {"M": M.clone()}
    yield "all None", (X, dims, [None] * 3, 1), {}
    yield "lam", (X, dims, A, 1), {"M": M.clone(), "lam": lam}
    yield "beta", (X, dims, A, 1), {"M": M.clone(), "lam": lam, "beta": 0.5}
    yield "whole beta", (X, dims, A, 1), {"M": M.clone(), "beta": 1}
    yield "workspace", (X, dims, A, 1), {"workspace": ws}
    yield "workspace, beta", (X, dims, A, 1), {"workspace": ws, "M": M.clone(), "beta": 2.0}
    yield "small workspace", (X, dims, A, 0), {"workspace": ws[:0]}
    yield "stream", (X, dims, A, 1), {"stream": torch.cuda.current_stream().cuda_stream}
    yield "gradients", (X.clone().requires_grad_(), dims, [torch.nn.Parameter(a) for a in A], 1), {}
    yield "subclass", (X.as_subclass(Sub), dims, A, 1), {}
    yield "negative mode", (X, dims, A, -1), {}
    yield "mode too high", (X, dims, A, 3), {}
    yield "one mode", (X[:6], (6,), A[:1], 0), {}
    yield "extent 0", (X[:0], (6, 0, 4), [A[0], A[1][:0], A[2]], 0), {}
    yield "no columns", (X, dims, [a[:, :0].contiguous() for a in A], 1), {}
    yield "wrong number of values", (X[:-1], dims, A, 1), {}
    yield "strided X", (torch.cat([X, X])[::2], dims, A, 1), {}
    yield "other type", (X, dims, [A[0].to(other), A[1], A[2]], 1), {}
    yield "half", (X.half(), dims, A, 1), {}
    yield "on the CPU", (X.cpu(), dims, A, 1), {}
    yield "factor on the CPU", (X, dims, [A[0].cpu(), A[1], A[2]], 1), {}
    yield "strided factor", (X, dims, [A[0], wide[:, :R], A[2]], 0), {}
    yield "ranks differ", (X, dims, [A[0], wide.contiguous(), A[2]], 0), {}
    yield "rows differ", (X, dims, [A[1], A[1], A[2]], 1), {}
    yield "factors missing", (X, dims, A[:2], 1), {}
    yield "strided M", (X, dims, A, 1), {"M": wide[:, :R]}
    yield "shape of M", (X, dims, A, 1), {"M": M[:4]}
    yield "type of M", (X, dims, A, 1), {"M": M.to(other)}
    yield "length of lam", (X, dims, A, 1), {"lam": lam[:2]}
    yield "type of lam", (X, dims, A, 1), {"lam": lam.to(other)}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_both_ways_agree(dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import os
    from paper_2510_14891_amd import binding as mt
    assert os.path.exists(mt.CALL_PATH)
    T = torch.float64 if dtype == "f64" else torch.float32
    pairs = list(zip(forms(T), forms(T)))          # each side has inputs of its own
    taken = 0
    for (name, args, kw), (_, args2, kw2) in pairs:
        print("dense call, form: %s" % name, flush=True)
        a, b = outcome(mt, True, args, kw), outcome(mt, False, args2, kw2)
        assert a[0] == b[0] and a[2] == b[2], (name, a, b)
        assert torch.equal(a[1], b[1]) if a[0] == "ok" else a[1] == b[1], (name, a, b)
        taken += a[0] == "ok"
    assert taken >= 14
