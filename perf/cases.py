"""Performance cases of the library: what its users run, through its public
entry points.

The listed cases are the steps of the solves that ``bench.py`` and the tests
run (the data pass of an iteration, the sketches, the metric factor, the
staging of reduced-precision copies, the sparse pass), at those workloads'
sizes and at the ragged sizes of the serving trace, and two whole solves.
``draw`` gives more of the same kinds over the same ranges.

Inputs follow the library's synthetic recipes (two views of one Gaussian
latent factor, columns scaled over decades; sparse rows with Zipf-like column
popularity), drawn on the device from the seed.  Products of FP32 and BF16
arithmetic come back as sums of that precision in doubles; the program here
keeps them, like the data they belong to, in FP32.
"""
import math

import numpy as np
import torch

import paper_2106_12060_amd as srp

DEV = "cuda"
TORCH = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"f64": 8, "f32": 4, "bf16": 2, "fp8": 1}


def listed():
    return [
        # one iteration's products of the FP64 CCA configuration: the
        # smallest call a solve makes, all latency
        {"name": "pass-f64-small", "op": "pass", "dtype": "f64", "n": 2000, "d0": 60, "d1": 40, "k": 5},
        # the same step for a typical request of the serving trace: mid-size,
        # row lengths that are no multiple of anything
        {"name": "pass-f32-ragged", "op": "pass", "dtype": "f32", "n": 52345, "d0": 531, "d1": 347, "k": 9},
        # the step that dominates the default benchmark (FP32 CCA)
        {"name": "pass-f32-cca", "op": "pass", "dtype": "f32", "n": 200000, "d0": 1000, "d1": 1000, "k": 10},
        # the FDA configuration's step: one view, all c - 1 directions
        {"name": "pass-f32-fda", "op": "pass", "dtype": "f32", "n": 100000, "d0": 2000, "d1": 0, "k": 19},
        # the reduced-precision CCA configuration's step
        {"name": "pass-bf16-cca", "op": "pass", "dtype": "bf16", "n": 200000, "d0": 1000, "d1": 1000, "k": 10},
        # one iteration's products of the sparse (bag-of-words-like) CCA
        # configuration
        {"name": "pass-csr", "op": "pass_csr", "n": 1000000, "d0": 1000, "d1": 1000, "k": 8, "per_row": 24},
        # preprocessing of the default benchmark: SRHT of one view
        {"name": "sketch-srht", "op": "sketch", "kind": "srht", "dtype": "f32", "n": 200000, "d": 1000, "s": 4000},
        # preprocessing of the FDA configuration: CountSketch
        {"name": "sketch-count", "op": "sketch", "kind": "count", "dtype": "f32", "n": 100000, "d": 2000, "s": 8000},
        # the metric of the default benchmark from its sketch
        {"name": "factor-cca", "op": "factor", "dtype": "f32", "s": 4000, "d": 1000},
        # staging one view of the reduced-precision configuration as FP8
        {"name": "stage-fp8", "op": "stage", "to": "fp8", "n": 200000, "d": 1000},
        # a whole request of the serving trace's kind, ragged, at its
        # tolerance: launches and small kernels count
        {"name": "solve-serving", "op": "solve", "sketch": "countsketch", "n": 20011, "d0": 301, "d1": 203, "k": 8,
         "r": 8, "decades": 3.0, "fdecades": 1.0, "tol": 1e-5},
        # the default benchmark itself
        {"name": "solve-cca", "op": "solve", "sketch": "srht", "n": 200000, "d0": 1000, "d1": 1000, "k": 10,
         "r": 32, "decades": 4.0, "fdecades": 2.0, "tol": 1e-4},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["pass", "pass", "pass", "pass", "sketch", "sketch", "factor", "stage", "pass_csr", "solve"])
    if op == "pass":
        dtype = rng.choice(["f64", "f32", "f32", "f32", "bf16"])
        if dtype == "f64":      # the FP64 pass takes up to 896 columns in all
            return {"op": op, "dtype": dtype, "n": _log(rng, 2000, 60000), "d0": _log(rng, 40, 448),
                    "d1": _log(rng, 40, 448), "k": rng.randint(2, 16)}
        if rng.random() < 0.3:  # FDA
            d = _log(rng, 200, 2048)
            d -= d % 4 if dtype == "bf16" else 0
            return {"op": op, "dtype": dtype, "n": _log(rng, 20 * d, 100000), "d0": d, "d1": 0,
                    "k": rng.randint(2, 19 if dtype == "f32" else 16)}
        d0, d1 = _log(rng, 64, 1024), _log(rng, 64, 1024)
        if dtype == "bf16":     # staged copies are read 4 bytes at a time
            d0, d1 = max(128, d0 - d0 % 2), max(128, d1 - d1 % 2)
        return {"op": op, "dtype": dtype, "n": _log(rng, max(5000, 20 * max(d0, d1)), 200000), "d0": d0, "d1": d1,
                "k": rng.randint(2, 16)}
    if op == "sketch":
        d = _log(rng, 64, 2000)
        return {"op": op, "kind": rng.choice(["srht", "count"]), "dtype": rng.choice(["f64", "f32", "f32", "fp8"]),
                "n": _log(rng, max(5000, 8 * d), 200000 if d <= 1000 else 100000), "d": d, "s": 4 * d}
    if op == "factor":
        d = _log(rng, 60, 2000)
        return {"op": op, "dtype": rng.choice(["f64", "f32", "f32"]), "s": 4 * d, "d": d}
    if op == "stage":
        return {"op": op, "to": rng.choice(["fp8", "bf16"]), "n": _log(rng, 5000, 200000), "d": _log(rng, 64, 1024)}
    if op == "pass_csr":
        return {"op": op, "n": _log(rng, 100000, 1000000), "d0": _log(rng, 200, 1000), "d1": _log(rng, 200, 1000),
                "k": rng.randint(2, 16), "per_row": rng.randint(8, 24)}
    d0, d1 = _log(rng, 64, 600), _log(rng, 64, 600)
    return {"op": op, "sketch": rng.choice(["countsketch", "srht"]), "n": _log(rng, 30 * max(d0, d1), 60000),
            "d0": d0, "d1": d1, "k": 8, "r": 8, "decades": 3.0, "fdecades": 1.0, "tol": 1e-5}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 12060)
    return g


def _randn(g, *shape, dtype=torch.float32):
    return torch.randn(shape, generator=g, device=DEV, dtype=dtype)


def _scales(d, decades):
    return torch.from_numpy(10.0 ** (-decades * np.arange(d) / d)).to(DEV)


def _views(g, n, dims, *, r=32, noise=1.0, decades=4.0, fdecades=2.0):
    """FP32 views of one latent factor, columns scaled over `decades`."""
    Z = _randn(g, n, r)
    Z.mul_((10.0 ** (-fdecades * torch.arange(r, device=DEV) / r)).float())
    out = []
    for d in dims:
        A = _randn(g, n, d)
        A.mul_(noise).addmm_(Z, _randn(g, r, d))
        out.append(A.mul_(_scales(d, decades).float()))
    return out


def _directions(g, n, d, k, decades=4.0):
    """Directions of an iterate's size: unit-variance products A W."""
    return _randn(g, d, k, dtype=torch.float64) / (_scales(d, decades) * math.sqrt(d))[:, None]


def _csr(g, n, d, per_row):
    """Poisson row lengths, column popularity (j + 1)^-0.7, 2 % of the rows
    empty, duplicates merged, columns ascending."""
    counts = torch.poisson(torch.full((n,), float(per_row), device=DEV), generator=g).long()
    counts[torch.rand(n, generator=g, device=DEV) < 0.02] = 0
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), counts)
    p = torch.arange(1, d + 1, device=DEV, dtype=torch.float64) ** -0.7
    cdf = torch.cumsum(p / p.sum(), 0)
    u = torch.rand(rows.numel(), generator=g, device=DEV, dtype=torch.float64)
    key = torch.unique(rows * d + torch.searchsorted(cdf, u).clamp_(max=d - 1))
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(torch.bincount(key // d, minlength=n), 0)
    return srp.Csr(ptr, (key % d).int().contiguous(), _randn(g, key.numel()), d)


def _fp8_codes(g, n, d):
    """E4M3 codes as the staging gives them (columns scaled to 448)."""
    return srp.srp_stage_fp8(_views(g, n, (d,))[0])[0]


def _inputs(case, seed):
    g = _gen(seed)
    op = case["op"]
    if op == "pass":
        dims = (case["d0"], case["d1"]) if case["d1"] else (case["d0"],)
        A = [a.to(TORCH[case["dtype"]]) for a in _views(g, case["n"], dims)]
        return A, [_directions(g, case["n"], d, case["k"]) for d in dims]
    if op == "pass_csr":
        dims = (case["d0"], case["d1"])
        A = [_csr(g, case["n"], d, case["per_row"]) for d in dims]
        return A, [_directions(g, case["n"], d, case["k"], 0.0) for d in dims]
    if op == "sketch":
        if case["dtype"] == "fp8":
            return _fp8_codes(g, case["n"], case["d"])
        return _views(g, case["n"], (case["d"],))[0].to(TORCH[case["dtype"]])
    if op == "factor":          # the sketch of 50 times as many rows
        return (_views(g, case["s"], (case["d"],))[0] * math.sqrt(50.0)).to(TORCH[case["dtype"]])
    if op == "stage":
        return _views(g, case["n"], (case["d"],))[0]
    return _views(g, case["n"], (case["d0"], case["d1"]), r=case["r"], decades=case["decades"],
                  fdecades=case["fdecades"])


LAMBDA = 1e-4      # of the factor and the solves
SKETCH_SEED = 12060


def prepare(case, seed):
    state = {"case": dict(case), "in": _inputs(case, seed)}
    if case["op"] == "solve":
        state["options"] = srp.srp_default_options(sketch=case["sketch"], max_iter=500, seed=SKETCH_SEED)
    return state


# --------------------------------------------------------------- one pass
def run(state):
    c, x = state["case"], state["in"]
    op = c["op"]
    if op == "pass":
        A, W = x
        second = (A[1], W[1]) if c["d1"] else ()
        J = srp.srp_gram_pass(A[0], W[0], *second, compute=c["dtype"])
        return [j if c["dtype"] == "f64" else j.float() for j in J if j is not None]
    if op == "pass_csr":
        A, W = x
        return list(srp.srp_gram_pass_csr(A[0], W[0], A[1], W[1]))
    if op == "sketch":
        return (srp.srp_srht if c["kind"] == "srht" else srp.srp_countsketch)(x, c["s"], SKETCH_SEED)
    if op == "factor":
        return list(srp.srp_sketch_factor(x, LAMBDA))
    if op == "stage":
        return list(srp.srp_stage_fp8(x)) if c["to"] == "fp8" else srp.srp_stage_bf16(x)
    U, V, sigma, _ = srp.cca_solve(x[0], x[1], c["k"], LAMBDA, LAMBDA, 4 * max(c["d0"], c["d1"]), tol=c["tol"],
                                   options=state["options"], mu=[1.0] * c["k"])
    return [U.float(), V.float(), sigma.float()]


def work(case):
    c, op = case, case["op"]
    if op == "pass":
        D, nb = c["d0"] + c["d1"], 2 if c["d1"] else 1
        return {"bytes": c["n"] * D * BYTES[c["dtype"]] + 8 * D * c["k"] * (1 + nb),
                "flops": 2 * (1 + nb) * c["n"] * D * c["k"]}
    if op == "pass_csr":        # an index and a value per entry
        nnz, D = c["n"] * c["per_row"] * 0.95, c["d0"] + c["d1"]
        return {"bytes": 2 * nnz * 8 + 16 * c["n"] + 24 * D * c["k"], "flops": 2 * 6 * nnz * c["k"]}
    if op == "sketch":
        out = 8 if c["dtype"] == "f64" else 4
        nd = c["n"] * c["d"]
        return {"bytes": nd * BYTES[c["dtype"]] + out * c["s"] * c["d"],
                "flops": nd * (1 if c["kind"] == "count" else math.log2(c["s"]))}
    if op == "factor":
        s, d = c["s"], c["d"]
        return {"bytes": s * d * BYTES[c["dtype"]] + 16 * d * d, "flops": s * d * d + 2 * d ** 3 / 3}
    if op == "stage":
        return {"bytes": c["n"] * c["d"] * (4 + BYTES[c["to"]]), "flops": c["n"] * c["d"]}
    D, s = c["d0"] + c["d1"], 4 * max(c["d0"], c["d1"])     # one read and one pass, and the metric
    return {"bytes": c["n"] * D * 4 + 8 * D * c["k"],
            "flops": 6 * c["n"] * D * c["k"] + sum(s * d * d + d ** 3 for d in (c["d0"], c["d1"]))}


# ------------------------------------------------------------- in 64 bits
def _splitmix64(seed, n):
    i = np.arange(1, n + 1, dtype=np.uint64)
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + i * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _signs(w):
    return torch.from_numpy(1.0 - 2.0 * (w & np.uint64(1)).astype(np.float64)).to(DEV)


def _exact_sketch(c, A):
    n, s = A.shape[0], c["s"]
    if c["dtype"] == "fp8":
        A = A.view(torch.float8_e4m3fn).float()
    out = []
    if c["kind"] == "count":
        w = _splitmix64(SKETCH_SEED, n)
        h = torch.from_numpy((((w >> np.uint64(32)) * np.uint64(s)) >> np.uint64(32)).astype(np.int64)).to(DEV)
        g = _signs(w)
        for j in range(0, A.shape[1], 256):
            B = A[:, j:j + 256].double() * g[:, None]
            out.append(torch.zeros(s, B.shape[1], dtype=torch.float64, device=DEV).index_add_(0, h, B))
    else:
        m = 2 if n < 2 else 1 << (n - 1).bit_length()
        key = _splitmix64(SKETCH_SEED ^ 0x535248545357524F, m)
        rows = torch.from_numpy(np.sort(np.argpartition(key, s - 1)[:s])).to(DEV)
        sign = _signs(_splitmix64(SKETCH_SEED ^ 0x5352485444494147, n))
        for j in range(0, A.shape[1], 128):
            B = A[:, j:j + 128].double() * sign[:, None]
            B = torch.cat([B, torch.zeros(m - n, B.shape[1], dtype=torch.float64, device=DEV)])
            q = 1
            while q < m:        # Walsh-Hadamard butterflies over the rows
                B = B.view(m // (2 * q), 2, q, -1)
                B = torch.stack([B[:, 0] + B[:, 1], B[:, 0] - B[:, 1]], 1).view(m, -1)
                q *= 2
            out.append(B[rows] / math.sqrt(s))
    return torch.cat(out, 1)


def _csr_mul(A, W):
    """A W and its transpose's product, entry by entry, in chunks."""
    n, d = A.shape
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), A.row_ptr.diff())
    P = torch.zeros(n, W.shape[1], dtype=torch.float64, device=DEV)
    for b in range(0, rows.numel(), 1 << 22):
        e = slice(b, b + (1 << 22))
        P.index_add_(0, rows[e], W[A.col_idx[e].long()] * A.values[e].double()[:, None])
    return rows, P


def _exact_solve(c, X, Y):
    X, Y = X.double(), Y.double()
    lam = torch.full((1,), LAMBDA, dtype=torch.float64, device=DEV)
    Rx, Ry = (torch.linalg.cholesky(A.T @ A + lam * torch.eye(A.shape[1], dtype=torch.float64, device=DEV)).cpu().numpy()
              for A in (X, Y))
    C = np.linalg.solve(Ry, np.linalg.solve(Rx, (X.T @ Y).cpu().numpy()).T).T
    P, sigma, Q = np.linalg.svd(C)
    k = c["k"]
    U, V = np.linalg.solve(Rx.T, P[:, :k]), np.linalg.solve(Ry.T, Q[:k].T)
    sign = np.sign(U[np.abs(U).argmax(0), np.arange(k)])
    return [torch.from_numpy(U * sign), torch.from_numpy(V * sign), torch.from_numpy(sigma[:k].copy())]


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    op = c["op"]
    if op == "pass":
        A, W = [a.double() for a in x[0]], x[1]
        P = torch.cat([a @ w for a, w in zip(A, W)], 1)
        return [a.T @ P for a in A]
    if op == "pass_csr":
        A, W = x
        m = [_csr_mul(a, w) for a, w in zip(A, W)]
        P = torch.cat([p for _, p in m], 1)
        J = []
        for a, (rows, _) in zip(A, m):
            j = torch.zeros(a.shape[1], P.shape[1], dtype=torch.float64, device=DEV)
            order = torch.argsort(a.col_idx.long(), stable=True)
            ends = torch.cumsum(torch.bincount(a.col_idx, minlength=a.shape[1]), 0).tolist()
            for col, (b, e) in enumerate(zip([0] + ends, ends)):
                q = order[b:e]
                j[col] = a.values[q].double() @ P[rows[q]]
            J.append(j)
        return J
    if op == "sketch":
        return _exact_sketch(c, x)
    if op == "factor":
        G = x.double().T @ x.double()
        G.diagonal().add_(LAMBDA)
        R = torch.linalg.cholesky(G).T.contiguous()
        inv = torch.linalg.solve_triangular(R, torch.eye(c["d"], dtype=torch.float64, device=DEV), upper=True)
        return [R, inv]
    if op == "stage":
        return None             # codes and powers of two, equal or wrong
    return _exact_solve(c, *x)
