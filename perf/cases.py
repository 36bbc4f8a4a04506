"""The work that users of this library have it do, as a list of cases for timing.

Callers are optimizers and solvers: a Muon-style step takes the polar factor of every weight gradient
(bf16, a few shapes, a small fixed number of iterations), a Shampoo-style step takes inverse roots of
its preconditioner statistics (fp32, to a tolerance), and the square roots, the matrix sign and the
inverse are called on single large matrices or small batches.  `listed()` names one case per kind of
call, from one 64 x 32 matrix to an 8192 x 8192 square root; `draw(rng)` gives more of the same kinds
over their whole range of sizes.

The library works in place, so a pass copies its input first, as a caller that keeps its gradients or
statistics does.  Inputs are synthetic: drawn on the GPU from the seed alone.
"""
import math

import torch

from paper_2601_22137_amd import optim, prism

SKETCH_SEED = 22137


# ------------------------------------------------------------------------------------------- cases

def listed():
    return [
        # One small fp32 polar factor to a tight tolerance: nothing but latency.
        {"name": "polar_f32_small", "kind": "polar_f32", "batch": 1, "m": 64, "n": 32, "degree": 5, "sketch": 8,
         "tol": 1e-6, "max_iters": 30},
        # A few fp32 matrices of ordinary, ragged size (a solver's subspaces): both sides odd against every tile.
        {"name": "polar_f32_ragged", "kind": "polar_f32", "batch": 6, "m": 500, "n": 299, "degree": 5, "sketch": 8,
         "tol": 1e-5, "max_iters": 40},
        # One weight gradient: the smallest bf16 call of a Muon-style step.
        {"name": "muon_one_weight", "kind": "muon", "layers": 1, "width": 768, "shapes": "wide", "iters": 5, "warm": 0},
        # The 2-D gradients of a stack of layers of width 768 (square, 4x wide, 4x tall, 3x wide), one call.
        {"name": "muon_layers_768", "kind": "muon", "layers": 16, "width": 768, "shapes": "block", "iters": 5, "warm": 0},
        # The paper's Muon setting: ten layers of width 1024, three iterations at the upper coefficient, no fit.
        {"name": "muon_layers_1024_warm", "kind": "muon", "layers": 10, "width": 1024, "shapes": "block", "iters": 3, "warm": 3},
        # Large square matrices over four decades of singular values to a tolerance, split iterate.
        {"name": "polar_bf16_large", "kind": "polar_bf16", "batch": 8, "m": 4096, "n": 4096, "decades": 4.0, "degree": 5,
         "sketch": 32, "tol": 1e-2, "max_iters": 40},
        # An embedding's gradient: one tall matrix whose row count no vector width divides.
        {"name": "polar_bf16_tall_ragged", "kind": "muon_tall", "m": 50257, "n": 768, "iters": 5},
        # Preconditioners of a small convolutional network: sizes from a few entries to a few hundred, mixed.
        {"name": "shampoo_small_mixed", "kind": "shampoo", "sizes": "27,16,144,16,144,32,288,32,288,64,576,64,576,64,64,10",
         "root_p": 4, "sketch": 16, "tol": 1e-5, "max_iters": 40},
        # Inverse fourth roots of a batch of large preconditioners.
        {"name": "inv_root_1024", "kind": "inv_root", "batch": 32, "n": 1024, "root_p": 4, "sketch": 16, "tol": 1e-5,
         "max_iters": 40},
        # Square root and inverse square root of one matrix of the largest size.
        {"name": "sqrt_8192", "kind": "sqrt", "batch": 1, "n": 8192, "degree": 5, "sketch": 64, "tol": 1e-5, "max_iters": 40},
        # The same by the Newton variant, at the largest preconditioner size of the paper's experiments.
        {"name": "sqrt_newton_2048", "kind": "sqrt_newton", "batch": 2, "n": 2048, "tol": 1e-5, "max_iters": 12},
        # Matrix sign of a few symmetric indefinite matrices of ragged size.
        {"name": "sign_1000", "kind": "sign", "batch": 4, "n": 1000, "degree": 5, "sketch": 32, "tol": 1e-5, "max_iters": 40},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, unit):
    """Log-uniform size; half of them multiples of `unit` (what models use), half any number."""
    v = _log_int(rng, lo, hi)
    return max(unit, v // unit * unit) if rng.random() < 0.5 else v


def draw(rng):
    kind = rng.choice(["polar_f32", "muon", "muon", "polar_bf16", "muon_tall", "shampoo", "inv_root", "sqrt",
                       "sqrt_newton", "sign", "inverse"])
    if kind == "polar_f32":
        # clearly rectangular, either way round: a square Gaussian has a condition number of its own
        small = rng.random() < 0.5  # everything fits 64 x 64
        long = _log_int(rng, 8, 64) if small else _size(rng, 80, 1024, 64)
        short = min(_log_int(rng, 4, 40) if small else _size(rng, 40, 600, 32), int(0.6 * long))
        m, n = (long, short) if rng.random() < 0.7 else (short, long)
        if small:
            return {"kind": kind, "batch": _log_int(rng, 1, 256), "m": m, "n": n, "degree": 5, "sketch": rng.choice([8, 16]),
                    "tol": 1e-6, "max_iters": 30}
        return {"kind": kind, "batch": _log_int(rng, 1, 16), "m": m, "n": n, "degree": rng.choice([3, 5]),
                "sketch": rng.choice([8, 16]), "tol": 1e-5, "max_iters": 40}
    if kind == "muon":
        width = _size(rng, 128, 1536, 64)
        warm = rng.random() < 0.3
        return {"kind": kind, "layers": _log_int(rng, 1, 16), "width": width, "shapes": rng.choice(["wide", "tall", "square", "block", "block"]),
                "iters": 3 if warm else 5, "warm": 3 if warm else 0}
    if kind == "polar_bf16":
        n = _size(rng, 512, 4096, 256)
        return {"kind": kind, "batch": rng.choice([1, 2, 4, 8]), "m": n + (0 if rng.random() < 0.5 else _log_int(rng, 8, 512)), "n": n,
                "decades": rng.choice([2.0, 4.0]), "degree": 5, "sketch": rng.choice([16, 32]), "tol": 1e-2, "max_iters": 40}
    if kind == "muon_tall":
        return {"kind": kind, "m": _log_int(rng, 8192, 65536), "n": _size(rng, 128, 1024, 64), "iters": 5}
    if kind == "shampoo":
        sizes = ",".join(str(_log_int(rng, 8, 640)) for _ in range(rng.randint(2, 16)))
        return {"kind": kind, "sizes": sizes, "root_p": rng.choice([2, 4]), "sketch": 16, "tol": 1e-5, "max_iters": 40}
    if kind == "inv_root":
        return {"kind": kind, "batch": _log_int(rng, 1, 32), "n": _size(rng, 256, 1024, 128), "root_p": rng.choice([2, 4]),
                "sketch": 16, "tol": 1e-5, "max_iters": 40}
    if kind == "sqrt":
        return {"kind": kind, "batch": rng.choice([1, 2, 4]), "n": _size(rng, 128, 4096, 128), "degree": 5,
                "sketch": rng.choice([16, 64]), "tol": 1e-5, "max_iters": 40}
    if kind == "sqrt_newton":
        return {"kind": kind, "batch": rng.choice([1, 2, 4]), "n": _size(rng, 256, 4096, 256), "tol": 1e-5, "max_iters": 12}
    if kind == "sign":
        return {"kind": kind, "batch": rng.choice([1, 2, 4, 8]), "n": _size(rng, 256, 2048, 128), "degree": rng.choice([3, 5]),
                "sketch": rng.choice([16, 32]), "tol": 1e-5, "max_iters": 40}
    return {"kind": "inverse", "batch": rng.choice([1, 2, 4, 8]), "n": _size(rng, 256, 2048, 128), "sketch": rng.choice([16, 32]),
            "tol": 1e-5, "max_iters": 40}


def _muon_shapes(case):
    w = case["width"]
    one = {"square": [(w, w)], "wide": [(w, 4 * w)], "tall": [(4 * w, w)],
           "block": [(w, w), (w, 4 * w), (4 * w, w), (w, 3 * w)]}[case["shapes"]]
    return [s for _ in range(case["layers"]) for s in one]


def _sizes(case):
    return [int(s) for s in case["sizes"].split(",")]


# ------------------------------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float32)


def _gradient(g, m, n):
    """Gaussian entries times a log-normal scale per row, Frobenius-normalised: a weight gradient's shape."""
    a = _randn(g, m, n) * torch.exp(_randn(g, m, 1))
    return (a / torch.linalg.norm(a)).to(torch.bfloat16)


def _orthonormal(g, n, k):
    """n x k with orthonormal columns: Cholesky QR in fp64, twice."""
    w = _randn(g, n, k).double()
    for _ in range(2):
        r = torch.linalg.cholesky(w.t() @ w)
        w = torch.linalg.solve_triangular(r, w.t().contiguous(), upper=False).t().contiguous()
    return w


def _reflect(w, x):
    """(I - 2 w w^T) x: a random reflection through a subspace of half the dimension mixes every coordinate."""
    return x - 2.0 * (w @ (w.t() @ x))


def _planted(g, m, n, sigmas):
    """fp32 [len(sigmas)][m][n], matrix b with the singular values sigmas[b] (m >= n)."""
    u, v = _orthonormal(g, m, max(1, n // 2)), _orthonormal(g, n, max(1, n // 2))
    out = torch.empty(len(sigmas), m, n, device="cuda")
    for b, s in enumerate(sigmas):
        d = torch.zeros(m, n, device="cuda", dtype=torch.float64)
        d[:n] = torch.diag(s.double())[torch.randperm(n, generator=g, device="cuda")]
        out[b] = _reflect(v, _reflect(u, d).t().contiguous()).t().float()
    return out


def _symmetric(g, n, lams):
    """fp32 [len(lams)][n][n] symmetric, matrix b with the eigenvalues lams[b]."""
    w = _orthonormal(g, n, max(1, n // 2))
    out = torch.empty(len(lams), n, n, device="cuda")
    for b, lam in enumerate(lams):
        d = torch.diag(lam.double()[torch.randperm(n, generator=g, device="cuda")])
        # a second, unequal mixing: one reflection of a diagonal alone is its own inverse
        p = torch.randperm(n, generator=g, device="cuda")
        a = _reflect(w, _reflect(w, d).t().contiguous())[p][:, p]
        a = _reflect(w, _reflect(w, a).t().contiguous())
        out[b] = (0.5 * (a + a.t())).float()
    return out


def _power_law(n):
    return torch.arange(1, n + 1, device="cuda", dtype=torch.float64) ** -1.5 + 1e-6


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "polar_f32":
        # Gaussian columns scaled over three decades (two for the larger ones)
        decades = 3.0 if case["tol"] < 5e-6 else 2.0
        m, n = max(case["m"], case["n"]), min(case["m"], case["n"])
        x = _randn(g, case["batch"], m, n) * 10.0 ** (-decades * _rand(g, case["batch"], 1, n))
        x = x if case["m"] >= case["n"] else x.transpose(1, 2)
        return {"case": case, "x": x.contiguous()}
    if kind == "muon":
        return {"case": case, "grads": [_gradient(g, m, n) for m, n in _muon_shapes(case)]}
    if kind == "muon_tall":
        return {"case": case, "x": _gradient(g, case["m"], case["n"])[None].contiguous()}
    if kind == "polar_bf16":
        sig = [10.0 ** (-case["decades"] * _rand(g, case["n"])) for _ in range(case["batch"])]
        return {"case": case, "x": _planted(g, case["m"], case["n"], sig).to(torch.bfloat16)}
    if kind == "shampoo":
        return {"case": case, "stats": [_symmetric(g, n, [_power_law(n)])[0] for n in _sizes(case)]}
    if kind == "inv_root":
        n = case["n"]
        return {"case": case, "x": _symmetric(g, n, [_power_law(n)] * case["batch"])}
    if kind in ("sqrt", "sqrt_newton"):
        n = case["n"]
        x = torch.empty(case["batch"], n, n, device="cuda")
        for b in range(case["batch"]):     # sample covariance with a ridge
            w = _randn(g, n, 2 * n)
            x[b] = (w @ w.t()) / (2.0 * n) + 1e-4 * torch.eye(n, device="cuda")
        return {"case": case, "x": x}
    n = case["n"]
    if kind == "sign":
        lam = [10.0 ** (-2.0 * _rand(g, n)) * torch.where(_rand(g, n) < 0.5, -1.0, 1.0) for _ in range(case["batch"])]
        return {"case": case, "x": _symmetric(g, n, lam)}
    sig = [torch.exp(-math.log(30.0) * _rand(g, n)) * (1.0 + 2.0 * b) for b in range(case["batch"])]
    return {"case": case, "x": _planted(g, n, n, sig)}


# -------------------------------------------------------------------------------------------- pass

def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "muon":
        return optim.muon_orthogonalize(state["grads"], 5, c["iters"], 16, SKETCH_SEED, warm_iters=c["warm"])
    if kind == "shampoo":
        return optim.shampoo_inverse_roots(state["stats"], c["root_p"], c["max_iters"], c["sketch"], SKETCH_SEED, c["tol"])[0]
    x = state["x"].clone()
    if kind == "muon_tall":
        prism.polar(x, 5, c["iters"], 16, SKETCH_SEED, 0.0, flags=prism.FLAG_BF16_PLAIN_ITERATE)
    elif kind in ("polar_f32", "polar_bf16"):
        prism.polar(x, c["degree"], c["max_iters"], c["sketch"], SKETCH_SEED, c["tol"])
    elif kind == "inv_root":
        prism.inv_root(x, c["root_p"], c["max_iters"], c["sketch"], SKETCH_SEED, c["tol"])
    elif kind == "sqrt":
        return [x, prism.sqrt(x, c["degree"], c["max_iters"], c["sketch"], SKETCH_SEED, c["tol"])[0]]
    elif kind == "sqrt_newton":
        return [x, prism.sqrt_newton(x, c["max_iters"], c["tol"])[0]]
    elif kind == "sign":
        prism.sign(x, c["degree"], c["max_iters"], c["sketch"], SKETCH_SEED, c["tol"])
    else:
        prism.inverse(x, c["max_iters"], c["sketch"], SKETCH_SEED, c["tol"])
    return x


# ------------------------------------------------------------------------------------ work, tolerance

def _iterations(case):
    """The fixed budget, or the iterations to the tolerance on these inputs (measured)."""
    if "iters" in case:
        return case["iters"]
    if case["kind"] == "polar_bf16":
        return 14 if case["decades"] > 3.0 else 8
    if case["kind"] in ("polar_f32", "sign"):
        return 9 if case["degree"] == 5 else 12
    return {"shampoo": 7, "inv_root": 8, "sqrt": 6, "sqrt_newton": 4, "inverse": 10}[case["kind"]]


def work(case):
    """Each input read once and each output written once; the dense products of the iterations, a
    product whose result is symmetric by construction (X^T X, the square of a symmetric matrix)
    counted by its upper half."""
    kind = case["kind"]
    k = _iterations(case)

    def polar(m, n):
        s, l = min(m, n), max(m, n)
        return k * (3.0 * l * s * s + (float(s) ** 3 if case.get("degree", 5) == 5 else 0.0))

    if kind in ("muon", "muon_tall"):
        shapes = _muon_shapes(case) if kind == "muon" else [(case["m"], case["n"])]
        return {"bytes": sum(4 * m * n for m, n in shapes), "flops": sum(polar(m, n) for m, n in shapes)}
    if kind in ("polar_f32", "polar_bf16"):
        size = 4 if kind == "polar_f32" else 2
        return {"bytes": 2 * size * case["batch"] * case["m"] * case["n"], "flops": case["batch"] * polar(case["m"], case["n"])}
    if kind in ("shampoo", "inv_root"):
        ns = _sizes(case) if kind == "shampoo" else [case["n"]] * case["batch"]
        # X R, the powers of I + alpha R up to p, their product with M
        per = (1.0 + 2.0 * math.ceil(math.log2(case["root_p"])) + 2.0)
        return {"bytes": sum(8 * n * n for n in ns), "flops": k * sum(per * float(n) ** 3 for n in ns)}
    n, b = case["n"], case["batch"]
    # square root: Y X, R^2, X Q, Q Y.  Newton: the inverse and two symmetric updates.  Sign, inverse: three products.
    per = {"sqrt": 8.0, "sqrt_newton": 4.0, "sign": 4.0 if case.get("degree", 5) == 3 else 6.0, "inverse": 6.0}[kind]
    outputs = 2 if kind in ("sqrt", "sqrt_newton") else 1
    return {"bytes": (1 + outputs) * 4 * b * n * n, "flops": k * b * per * float(n) ** 3}


def tolerance(case):
    """Measured against the same iterations carried out in fp64 with the reported coefficients (bf16, fp32
    polar) or against the eigendecomposition: bf16 4e-3 to 6e-3, fp32 polar 1e-7 to 5e-7, inverse roots
    1e-7 to 4e-6, square roots 2e-7 to 5e-7, sign and inverse 1e-6 to 3e-6; about four times that.  Runs to
    a tolerance leave room for a stop that rounding decides (the last update moves the result by at
    most half the tolerance)."""
    return {"rel": {"polar_f32": 5e-6, "muon": 2e-2, "muon_tall": 2e-2, "polar_bf16": 2e-2, "shampoo": 1e-5, "inv_root": 1e-5,
                    "sqrt": 2e-6, "sqrt_newton": 2e-6, "sign": 1e-5, "inverse": 1e-5}[case["kind"]]}
