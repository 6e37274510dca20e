"""The workloads whose time this framework answers for, through its public entry points.

A case names a call, the tensor's extents, the data type, the rank and how X is made:

  mode          one MTTKRP (`mttkrp_dense`) of mode `k` into a buffer the program keeps
  modes         one MTTKRP per mode, d calls of `mttkrp_dense` on the same resident X
  shared        all modes from two passes over X (`mttkrp_dense_all_modes_shared`)
  cpals         `sweeps` sweeps of CP-ALS from a given start, every MTTKRP a pass of its own
  cpals_shared  the same with the modes of a sweep sharing partial contractions

`weighted` calls pass the weight vector lambda and accumulate into M (beta = 1).
"""
from __future__ import annotations

import math

import torch

from paper_2510_14891_amd import binding as mt

DTYPES = {"f64": torch.float64, "f32": torch.float32}


def listed():
    return [
        # The smallest call: a 2 MB tensor that stays in cache; launches and their gaps are what counts.
        dict(name="modes_64x64x64_f64_R16", call="modes", dims="64x64x64", dtype="f64", rank=16, x="uniform"),
        # An everyday decomposition: a 4 MB data set, low rank, a dozen sweeps.
        dict(name="cpals_100x80x60_f64_R10", call="cpals", dims="100x80x60", dtype="f64", rank=10, x="kruskal", sweeps=12),
        # Three long modes, the ordinary three-way tensor (4 GiB), every mode for itself and then the whole
        # sweep as a CP program asks for it.
        dict(name="modes_1024x1024x512_f64_R32", call="modes", dims="1024x1024x512", dtype="f64", rank=32, x="normal"),
        dict(name="shared_1024x1024x512_f64_R32", call="shared", dims="1024x1024x512", dtype="f64", rank=32, x="normal"),
        # Single precision, five equal modes, a rank at which the matrix cores count.
        dict(name="modes_48x48x48x48x48_f32_R64", call="modes", dims="48x48x48x48x48", dtype="f32", rank=64, x="kruskal"),
        # Many short modes of different extents (288 MB).
        dict(name="modes_20x30x40x50x60_f64_R16", call="modes", dims="20x30x40x50x60", dtype="f64", rank=16, x="uniform"),
        # One very long mode before two short ones: samples by small feature maps, single precision.
        dict(name="modes_1000000x20x20_f32_R32", call="modes", dims="1000000x20x20", dtype="f32", rank=32, x="normal"),
        # The largest tensor (16 GiB) at a rank above one pass of output columns, its middle mode.
        dict(name="mode_16384x2048x64_f64_R128_k1", call="mode", dims="16384x2048x64", dtype="f64", rank=128, k=1, x="uniform"),
        # Odd extents that no tile divides and a rank in the hundreds, first mode, with weights and accumulation.
        dict(name="mode_401x201x12x501_f64_R1000_k0", call="mode", dims="401x201x12x501", dtype="f64", rank=1000, k=0, x="uniform", weighted=True),
        # Odd extents, five-way (8 GB), low rank: every mode, and CP-ALS as it is run on such data.
        dict(name="modes_129x129x129x12x39_f64_R10", call="modes", dims="129x129x129x12x39", dtype="f64", rank=10, x="kruskal"),
        dict(name="cpals_shared_129x129x129x12x39_f64_R10", call="cpals_shared", dims="129x129x129x12x39", dtype="f64", rank=10, x="kruskal", sweeps=4),
        # CP-ALS at a rank in the hundreds on a 200 MB tensor.
        dict(name="cpals_129x129x129x12_f64_R500", call="cpals", dims="129x129x129x12", dtype="f64", rank=500, x="kruskal", sweeps=2),
    ]


def _dims(case):
    return tuple(int(v) for v in case["dims"].split("x"))


def _passes(case):
    """Passes over X a call of this kind needs: one per mode for separate calls; two per sweep where the
    modes may share partial contractions, as any iteration over the modes can do."""
    d = len(_dims(case))
    if case["call"] == "mode":
        return 1
    if case["call"] == "modes":
        return d
    return min(2, d) * case.get("sweeps", 1)


def work(case):
    dims, R = _dims(case), case["rank"]
    N, s = math.prod(dims), 8 if case["dtype"] == "f64" else 4
    p = _passes(case)
    return {"bytes": float(p * s * (N + R * sum(dims))), "flops": float(p * 2 * N * R)}


# No drawn case costs more than this (bytes, or flops / 50): that of the 16 GiB tensor above.
_MOST = 1.7e10


def draw(rng):
    """Another case of the same ranges: 3 to 6 modes (balanced, one long mode first, middle or last, short
    modes, odd extents), 2^18 to 2^31 values, ranks 4 to 128 and a few in the hundreds, both types."""
    while True:
        call = rng.choice(["mode", "mode", "modes", "modes", "modes", "shared", "cpals", "cpals_shared"])
        d = rng.choice([3, 3, 3, 4, 4, 5, 6])
        log_n = rng.uniform(18.0, 31.0)
        style = rng.choice(["balanced", "balanced", "spread", "long"])
        if style == "balanced":
            w = [rng.uniform(0.8, 1.25) for _ in range(d)]
        elif style == "spread":
            w = [rng.uniform(0.4, 1.6) for _ in range(d)]
        else:
            w = [1.0] * d
            w[rng.randrange(d)] = 1.3 * d
        dims = [max(3, round(2.0 ** (log_n * v / sum(w)))) for v in w]
        if rng.random() < 0.3:
            dims = [max(8, 8 * round(v / 8)) for v in dims]
        case = dict(call=call, dims="x".join(str(v) for v in dims), dtype="f64", rank=round(2.0 ** rng.uniform(2.0, 7.0)),
                    x=rng.choice(["uniform", "normal"]))
        if call in ("mode", "modes", "shared"):
            case["dtype"] = rng.choice(["f64", "f64", "f32"])
        if call == "mode":
            case["k"] = rng.randrange(d)
            if rng.random() < 0.25:
                case["rank"] = round(2.0 ** rng.uniform(7.0, 10.0))
            if rng.random() < 0.25:
                case["weighted"] = True
        N = math.prod(dims)
        if call == "shared":
            # two intermediates of (P + N / P) rows beside X: the shapes a program has that calls this
            case["rank"] = min(case["rank"], 48)
            cut = min(math.prod(dims[:s]) + N // math.prod(dims[:s]) for s in range(1, d))
            if N < 2 ** 27 or 4 * cut * case["rank"] > N // 16:
                continue
        if call.startswith("cpals"):
            case["x"] = "kruskal"
            case["sweeps"] = rng.randint(2, 4 if N > 2 ** 24 else 12)
            # a decomposition's rank: below every mode's number of other entries, and of its longer modes
            case["rank"] = min(case["rank"], sorted(dims)[1])
            if max(dims) > 200000:
                continue
        w = work(case)
        if max(w["bytes"], w["flops"] / 50) <= _MOST and N >= 2 ** 17:
            return case


def _fill(out, kind, gen):
    flat = out.view(-1)
    step = 1 << 28
    for i in range(0, flat.numel(), step):
        part = flat[i:i + step]
        if kind == "uniform":
            part.uniform_(0.0, 1.0, generator=gen)
        else:
            part.normal_(0.0, 1.0, generator=gen)
    return out


def _krp(factors):
    """Khatri-Rao product of the factors, lowest mode fastest: (prod I_m) x R."""
    K = factors[0]
    for A in factors[1:]:
        K = (A[:, None, :] * K[None, :, :]).reshape(-1, K.shape[1])
    return K


def _kruskal(dims, S, gen, dtype):
    """A rank-S tensor plus 1 % of noise, what a decomposition is run on; flat, first index fastest."""
    A = [_fill(torch.empty((I, S), dtype=torch.float64, device="cuda"), "normal", gen) for I in dims]
    X = torch.empty(math.prod(dims), dtype=dtype, device="cuda")
    s = (len(dims) + 1) // 2
    low, high = _krp(A[:s]), _krp(A[s:])
    Q = X.view(high.shape[0], low.shape[0])
    step = max(1, (1 << 27) // low.shape[0])
    for i in range(0, Q.shape[0], step):
        part = high[i:i + step] @ low.t()
        part += 0.01 * math.sqrt(S) * torch.randn(part.shape, dtype=part.dtype, device="cuda", generator=gen)
        Q[i:i + step] = part.to(dtype)
    return X


def prepare(case, seed):
    """X, the factors and the result buffers on the GPU."""
    dims, R, dtype = _dims(case), case["rank"], DTYPES[case["dtype"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["x"] == "kruskal":
        # decompositions run at the rank of their data, from nonnegative starts
        als = case["call"].startswith("cpals")
        X = _kruskal(dims, R if als else 8, gen, dtype)
        dist = "uniform" if als else "normal"
    else:
        X = _fill(torch.empty(math.prod(dims), dtype=dtype, device="cuda"), case["x"], gen)
        dist = case["x"]
    A = [_fill(torch.empty((I, R), dtype=dtype, device="cuda"), dist, gen) for I in dims]
    state = dict(case=case, dims=dims, X=X, A=A)
    if case["call"] == "mode":
        state["M"] = torch.empty((dims[case["k"]], R), dtype=dtype, device="cuda")
        if case.get("weighted"):
            state["lam"] = _fill(torch.empty(R, dtype=dtype, device="cuda"), "uniform", gen)
            state["M0"] = _fill(torch.empty_like(state["M"]), "normal", gen)
    elif not case["call"].startswith("cpals"):
        state["M"] = [torch.empty((I, R), dtype=dtype, device="cuda") for I in dims]
    torch.cuda.synchronize()
    return state


def run(state):
    case, dims, X, A = state["case"], state["dims"], state["X"], state["A"]
    call = case["call"]
    if call == "mode":
        if case.get("weighted"):
            M = state["M"].copy_(state["M0"])
            return mt.mttkrp_dense(X, dims, A, case["k"], M=M, lam=state["lam"], beta=1.0)
        return mt.mttkrp_dense(X, dims, A, case["k"], M=state["M"])
    if call == "modes":
        return [mt.mttkrp_dense(X, dims, A, k, M=state["M"][k]) for k in range(len(dims))]
    if call == "shared":
        return mt.mttkrp_dense_all_modes_shared(X, dims, A, M_out=state["M"])
    factors = [a.clone() for a in A]
    lam, fits = mt.mttkrp_cpals(X, dims, factors, case["sweeps"], 0.0, shared=call == "cpals_shared")
    return {"factors": factors, "lambda": lam, "fits": fits}


def tolerance(case):
    """Relative errors between correct implementations: about four times what these sums in another order
    (matrix products in 64 bits) showed over the listed and sixty drawn cases."""
    if case["call"].startswith("cpals"):
        # rounding times the condition of every sweep's normal equations: 1e-14 to 1e-9 seen, by the data
        return {"rel": 1e-7, "max": 1e-6}
    if case["dtype"] == "f64":
        return {"rel": 1e-12, "max": 1e-11}       # seen: 2e-13 and 8e-13, where sums of both signs cancel
    return {"rel": 5e-6, "max": 5e-5}             # seen: 1.1e-6 and 5e-6


def _mttkrp64(X, dims, A, k):
    """X_(k) times the Khatri-Rao product of the other factors, in float64 by matrix products."""
    R = next(a for m, a in enumerate(A) if m != k).shape[1]
    P, Q, Ik = math.prod(dims[:k]), math.prod(dims[k + 1:]), dims[k]
    M = torch.zeros((Ik, R), dtype=torch.float64, device=X.device)
    low = _krp([A[m].double() for m in range(k)]) if k > 0 else None
    high = _krp([A[m].double() for m in range(k + 1, len(dims))]) if k + 1 < len(dims) else None
    if low is None:
        step = max(1, (1 << 27) // Ik)
        for q in range(0, Q, step):
            M += X.view(Q, Ik)[q:q + step].double().t() @ high[q:q + step]
        return M
    if high is None:
        step = max(1, (1 << 27) // P)
        for i in range(0, Ik, step):
            M[i:i + step] = X.view(Ik, P)[i:i + step].double() @ low
        return M
    step = max(1, (1 << 27) // (Ik * max(P, R)))
    for q in range(0, Q, step):
        part = X.view(Q, Ik * P)[q:q + step].double().reshape(-1, P) @ low
        M += (part.view(-1, Ik, R) * high[q:q + step, None, :]).sum(0)
    return M


def exact(case, seed):
    state = prepare(case, seed)
    dims, X, A = state["dims"], state["X"], state["A"]
    call = case["call"]
    if call == "mode":
        M = _mttkrp64(X, dims, A, case["k"])
        return M * state["lam"].double() + state["M0"].double() if case.get("weighted") else M
    if not call.startswith("cpals"):
        return [_mttkrp64(X, dims, A, k) for k in range(len(dims))]
    A = [a.clone() for a in A]
    G = [a.t() @ a for a in A]
    norm2 = float((X * X).sum())
    fits = []
    for _ in range(case["sweeps"]):
        for k in range(len(dims)):
            M = _mttkrp64(X, dims, A, k)
            V = torch.ones_like(G[0])
            for m in range(len(dims)):
                if m != k:
                    V = V * G[m]
            A[k] = torch.cholesky_solve(M.t().contiguous(), torch.linalg.cholesky(V)).t().contiguous()
            lam = A[k].norm(dim=0)
            A[k] = A[k] / lam
            G[k] = A[k].t() @ A[k]
        V = torch.ones_like(G[0])
        for g in G:
            V = V * g
        inner = float((lam * (M * A[-1]).sum(0)).sum())
        fits.append(1.0 - math.sqrt(max(norm2 + float(lam @ V @ lam) - 2.0 * inner, 0.0)) / math.sqrt(norm2))
    return {"factors": A, "lambda": lam, "fits": fits}
