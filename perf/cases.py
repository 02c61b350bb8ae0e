"""The work a user of this library has it do, as cases that can be timed: whole trainings (tron_solve, tron_batch_solve),
the evaluation calls a caller with a trust-region loop of its own makes (tron_fun_grad, tron_hv, tron_hess_diag and their
multi-problem forms), and a training that starts from host arrays.  Sparse and dense, both losses, from problems that
finish in a fraction of a millisecond to a matrix of 44 GB.  Everything is fp64, the only type the library computes in.

Inputs are drawn on the GPU from the seed: sparse rows with uniform or Zipf-distributed columns and lognormal or binary
values scaled to unit length, dense rows from two Gaussians at +-mu (|mu| = 0.5); labels from a noisy planted model."""
import math

import numpy as np
import torch

import paper_2008_03433_amd as tron

LR, SVM = 0, 1

#: (function and gradient evaluations, Hessian-vector products) of a solve at eps = 0.01 on inputs of each kind, for work();
#: sparse inputs with uniform columns take about as many as dense ones
SOLVE_PASSES = {"sparse_solve": (5, 28), "sparse_train": (5, 24), "dense_solve": (3, 2), "batch_solve": (3, 2)}


def listed():
    return [
        # the smallest sparse training: 100,000 nonzeros, a few iterations; launches and waits count
        {"name": "sparse_solve_2k", "kind": "sparse_solve", "n": 2000, "d": 5000, "mean": 50, "zipf": 0.0, "lengths": "const", "values": "lognormal",
         "loss": LR, "C": 1.0, "blend": 0.0},
        # text classification, rcv1 shape: Poisson rows, Zipf features with tf-idf-like values
        {"name": "sparse_solve_rcv1", "kind": "sparse_solve", "n": 20242, "d": 47236, "mean": 74, "zipf": 1.1, "lengths": "poisson", "values": "lognormal",
         "loss": LR, "C": 1.0, "blend": 0.0},
        # the same shape as a program trains it once: host arrays in, preconditioned solve, weights back on the host
        {"name": "sparse_train_host", "kind": "sparse_train", "n": 20242, "d": 47236, "mean": 74, "zipf": 1.1, "lengths": "poisson", "values": "lognormal",
         "loss": LR, "C": 1.0, "blend": 0.01},
        # url shape, 123M nonzeros, binary features scaled per row: one gradient and the products of an inner solve
        {"name": "sparse_calls_url", "kind": "sparse_calls", "n": 2_000_000, "d": 3_000_000, "mean": 115, "zipf": 1.2, "lengths": "geometric", "values": "binary",
         "loss": LR, "C": 1.0, "products": 4, "diag": False},
        # a large matrix with free values (tf-idf), L2-SVM, with the Hessian diagonal a preconditioned loop asks for
        {"name": "sparse_calls_values", "kind": "sparse_calls", "n": 500_000, "d": 750_000, "mean": 80, "zipf": 1.1, "lengths": "poisson", "values": "lognormal",
         "loss": SVM, "C": 1.0, "products": 4, "diag": True},
        # a small set of dense feature vectors (peptide matches: 24 features), the usual interactive size
        {"name": "dense_solve_20k", "kind": "dense_solve", "n": 20_000, "d": 24, "loss": SVM, "C": 0.1},
        # dense L2-SVM, a million rows of 24 features
        {"name": "dense_solve_1m", "kind": "dense_solve", "n": 1_000_000, "d": 24, "loss": SVM, "C": 0.1},
        # dense logistic regression, 5M x 18
        {"name": "dense_solve_lr_5m", "kind": "dense_solve", "n": 5_000_000, "d": 18, "loss": LR, "C": 1.0},
        # wide dense rows, an odd number of columns
        {"name": "dense_calls_wide", "kind": "dense_calls", "n": 200_003, "d": 257, "loss": LR, "C": 1.0, "products": 2, "w_norm": 0.5, "diag": True},
        # the largest dense matrix, 44 GB
        {"name": "dense_calls_230m", "kind": "dense_calls", "n": 230_000_000, "d": 24, "loss": SVM, "C": 0.1, "products": 2, "w_norm": 0.2, "diag": False},
        # cross-validation: three folds x two C values, trained together
        {"name": "batch_solve_cv6", "kind": "batch_solve", "n": 1_000_000, "d": 24, "loss": SVM, "folds": 3, "Cs": 2},
        # nested cross-validation with logistic loss, twelve problems: one evaluation and the products of an inner solve
        {"name": "batch_calls_cv12", "kind": "batch_calls", "n": 20_000_000, "d": 24, "loss": LR, "folds": 3, "Cs": 4, "products": 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "text", "train", "url", "values", "dense", "dense", "dense_lr", "wide", "tall", "cv", "cv_calls"])
    if kind == "small":
        return {"kind": "sparse_solve", "n": _log(rng, 500, 8000), "d": _log(rng, 1000, 20000), "mean": rng.randint(10, 80), "zipf": 0.0,
                "lengths": rng.choice(["const", "poisson"]), "values": rng.choice(["lognormal", "binary"]), "loss": LR, "C": rng.choice([0.5, 1.0, 2.0]),
                "blend": rng.choice([0.0, 0.0, 0.01])}
    if kind in ("text", "train"):
        # C falls with the number of rows, as a user who tunes it finds: the inner solves stay at some tens of products
        n = _log(rng, 8000, 80000)
        return {"kind": "sparse_solve" if kind == "text" else "sparse_train", "n": n, "d": int(n * rng.uniform(1.5, 4.0)), "mean": rng.randint(40, 80),
                "zipf": round(rng.uniform(1.02, 1.12), 3), "lengths": "poisson", "values": rng.choice(["lognormal", "lognormal", "binary"]), "loss": LR,
                "C": round(min(1.0, 2e4 / n) * rng.choice([0.25, 0.5, 1.0]), 4), "blend": rng.choice([0.0, 0.0, 0.01]) if kind == "text" else rng.choice([0.0, 0.01])}
    if kind in ("url", "values"):
        n = _log(rng, 300_000, 2_000_000) if kind == "url" else _log(rng, 150_000, 600_000)
        return {"kind": "sparse_calls", "n": n, "d": int(n * rng.uniform(1.0, 1.5)), "mean": rng.randint(60, 115) if kind == "url" else rng.randint(40, 80),
                "zipf": round(rng.uniform(1.1, 1.2) if kind == "url" else rng.uniform(1.05, 1.15), 3), "lengths": "geometric" if kind == "url" else "poisson",
                "values": "binary" if kind == "url" else "lognormal", "loss": rng.choice([LR, SVM]), "C": 1.0, "products": rng.randint(2, 4),
                "diag": rng.random() < 0.5}
    if kind == "dense":
        return {"kind": "dense_solve", "n": _log(rng, 2000, 3_000_000), "d": rng.randint(4, 32), "loss": SVM, "C": rng.choice([0.1, 0.3, 1.0])}
    if kind == "dense_lr":
        return {"kind": "dense_solve", "n": _log(rng, 100_000, 6_000_000), "d": rng.randint(8, 32), "loss": LR, "C": rng.choice([0.3, 1.0])}
    if kind == "wide":
        return {"kind": "dense_calls", "n": _log(rng, 20_000, 250_000), "d": _log(rng, 33, 512), "loss": rng.choice([LR, SVM]), "C": 1.0,
                "products": rng.randint(1, 3), "w_norm": 0.5, "diag": rng.random() < 0.5}
    if kind == "tall":
        d = rng.randint(10, 28)
        return {"kind": "dense_calls", "n": _log(rng, 5_000_000, 5_000_000_000 // d), "d": d, "loss": rng.choice([LR, SVM]), "C": 0.1, "products": 2,
                "w_norm": rng.choice([0.2, 1.0, 3.0]), "diag": False}
    if kind == "cv":
        return {"kind": "batch_solve", "n": _log(rng, 50_000, 3_000_000), "d": rng.randint(8, 32), "loss": SVM, "folds": 3, "Cs": rng.randint(1, 3)}
    return {"kind": "batch_calls", "n": _log(rng, 1_000_000, 15_000_000), "d": rng.randint(8, 32), "loss": rng.choice([LR, SVM]), "folds": 3,
            "Cs": rng.randint(1, 5), "products": 2}


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, dtype=torch.float64, device="cuda")


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, dtype=torch.float64, device="cuda")


def _column_weights(case):
    ranks = torch.arange(1, case["d"] + 1, dtype=torch.float64, device="cuda")
    p = ranks.pow(-case["zipf"])
    return p / p.sum()


def _sparse(case, g):
    """(rowptr, col, val, y) on the GPU: draws per row, repeated columns dropped."""
    n, d, mean = case["n"], case["d"], case["mean"]
    if case["lengths"] == "const":
        draws = torch.full((n,), mean, dtype=torch.int64, device="cuda")
    elif case["lengths"] == "poisson":
        draws = torch.poisson(torch.full((n,), float(mean), dtype=torch.float64, device="cuda"), generator=g).to(torch.int64).clamp_(min=1)
    else:
        draws = (torch.log(1.0 - _uniform(g, n)) / math.log(1.0 - 1.0 / mean)).to(torch.int64).add_(1).clamp_(max=2000)
    total = int(draws.sum())
    if case["zipf"] > 0.0:
        edges = torch.cumsum(_column_weights(case).cpu(), 0).cuda()
        cols = torch.searchsorted(edges, _uniform(g, total)).clamp_(max=d - 1)
        cols = torch.randperm(d, generator=g, device="cuda")[cols]
    else:
        cols = torch.randint(d, (total,), generator=g, device="cuda")
    key = torch.repeat_interleave(torch.arange(n, device="cuda") * d, draws) + cols
    del cols
    key = torch.sort(key).values
    keep = torch.ones_like(key, dtype=torch.bool)
    torch.ne(key[1:], key[:-1], out=keep[1:])
    key = key[keep]
    del keep
    row = torch.div(key, d, rounding_mode="floor")
    col = (key - row * d).to(torch.int32)
    del key
    counts = torch.bincount(row, minlength=n)
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(counts, 0, out=rowptr[1:])
    if case["values"] == "lognormal":
        val = torch.exp(_normal(g, col.numel()))
        scale = torch.segment_reduce(val * val, "sum", lengths=counts, initial=0.0).sqrt_().reciprocal_()
        val.mul_(scale[row])
    else:
        val = counts.to(torch.float64).sqrt_().reciprocal_()[row]
    planted = _normal(g, d)
    if case["values"] == "binary":
        planted.mul_(_uniform(g, d) < 0.01 if d > 100_000 else 1.0)
    score = torch.segment_reduce(val * planted[col.to(torch.int64)], "sum", lengths=counts, initial=0.0)
    score += 0.1 * score.std() * _normal(g, n)
    y = torch.where(score >= score.median(), 1.0, -1.0).to(torch.float64)
    return rowptr, col, val, y


def _dense(case, g, stream_rows=4_000_000):
    """A handle of the matrix, written in chunks of rows, and the direction between the classes."""
    n, d = case["n"], case["d"]
    mu = _normal(g, d)
    mu *= 0.5 / mu.norm()
    scale = (1.0 + mu * mu).rsqrt()
    handle = tron.tron_dataset_create_dense_empty(n, d)
    for row0 in range(0, n, stream_rows):
        m = min(stream_rows, n - row0)
        side = torch.where(torch.arange(row0, row0 + m, device="cuda") % 2 == 0, 1.0, -1.0).to(torch.float64)
        X = _normal(g, m, d)
        X.addcmul_(side[:, None], mu[None, :]).mul_(scale)
        y = torch.where(_uniform(g, m) < 0.1, -side, side)
        tron.tron_dataset_write_rows(handle, row0, m, X, y)
    return tron.Dataset(handle), mu / mu.norm()


def _problems(case):
    return case["folds"] * case["Cs"]


def prepare(case, seed):
    g = _generator(seed)
    kind, d = case["kind"], case["d"]
    s = {"case": case}
    if kind.startswith("sparse"):
        rowptr, col, val, y = _sparse(case, g)
        if kind == "sparse_train":
            s["arrays"] = [t.cpu().numpy() for t in (rowptr, col, val, y)]
            return s
        s["data"] = tron.Dataset.from_csr(case["n"], d, rowptr, col, val, y)
        s["w"] = 0.5 * _normal(g, d)
    else:
        s["data"], along = _dense(case, g)
        s["w"] = case.get("w_norm", 0.0) * along
    if kind.startswith("batch"):
        K = _problems(case)
        fold = torch.randint(case["folds"], (case["n"],), generator=g, device="cuda", dtype=torch.int32)
        member = torch.zeros(case["n"], dtype=torch.int32, device="cuda")
        for k in range(K):
            member |= (fold != k % case["folds"]).to(torch.int32) << k
        s["batch"] = tron.Batch(s["data"], K, member)
        s["C"] = [float(0.03 * math.sqrt(10.0) ** (k // case["folds"])) for k in range(K)]
        s["W"] = 0.2 * along + 0.02 * _normal(g, K, d)
        s["V"] = [_normal(g, K, d) for _ in range(case.get("products", 0))]
        s["G"], s["HV"] = torch.empty_like(s["W"]), [torch.empty_like(v) for v in s["V"]]
    elif kind.endswith("calls"):
        s["V"] = [_normal(g, d) for _ in range(case["products"])]
        s["g"], s["HV"] = torch.empty_like(s["w"]), [torch.empty_like(s["w"]) for _ in s["V"]]
        s["diag"] = torch.empty_like(s["w"]) if case["diag"] else None
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------ one pass
def _trained(r, w):
    return {"w": w, "f": r.f, "outer": r.outer_iters, "products": r.cg_iters_total}


def run(s):
    case = s["case"]
    kind, loss = case["kind"], case["loss"]
    if kind == "sparse_train":
        rowptr, col, val, y = s["arrays"]
        data = tron.Dataset.from_csr(case["n"], case["d"], rowptr, col, val, y)
        w = torch.zeros(case["d"], dtype=torch.float64, device="cuda")
        r = data.solve(loss, case["C"], 0.01, w, precond_blend=case["blend"])
        data.close()
        return _trained(r, w.cpu())
    data = s["data"]
    if kind in ("sparse_solve", "dense_solve"):
        w = torch.zeros(case["d"], dtype=torch.float64, device="cuda")
        return _trained(data.solve(loss, case["C"], 0.01, w, precond_blend=case.get("blend", 0.0)), w)
    if kind == "batch_solve":
        W = torch.zeros_like(s["W"])
        r = s["batch"].solve(loss, s["C"], 0.01, W)
        return {"W": W, "f": [x.f for x in r], "outer": [x.outer_iters for x in r]}
    if kind == "batch_calls":
        f = s["batch"].fun_grad(loss, s["C"], s["W"], s["G"])
        curvature = [s["batch"].hv(s["C"], v, hv) for v, hv in zip(s["V"], s["HV"])]
        return {"f": np.array(f), "G": s["G"], "HV": s["HV"], "curvature": np.array(curvature)}
    f = data.fun_grad(loss, case["C"], s["w"], s["g"])
    if s["diag"] is not None:
        data.hess_diag(case["C"], s["diag"])
    curvature = [data.hv(case["C"], v, hv) for v, hv in zip(s["V"], s["HV"])]
    return {"f": f, "g": s["g"], "diag": s["diag"], "HV": s["HV"], "curvature": curvature}


# ------------------------------------------------------------------ what a pass cannot do without
def _nonzeros(case):
    """Expected nonzeros: a column of probability p is in a row of m draws unless all m miss it."""
    p = np.arange(1, case["d"] + 1, dtype=np.float64) ** -case["zipf"]
    p /= p.sum()
    m = float(case["mean"])
    if case["lengths"] == "const":
        hit = -np.expm1(m * np.log1p(-p))
    elif case["lengths"] == "poisson":
        hit = -np.expm1(-m * p)
    else:
        hit = m * p / (1.0 + (m - 1.0) * p)
    return case["n"] * float(hit.sum())


def work(case):
    n, d, kind = float(case["n"]), float(case["d"]), case["kind"]
    if kind.endswith("calls"):
        funs, products, diags = 1, case["products"], 1 if case.get("diag") else 0
    else:
        (funs, products), diags = SOLVE_PASSES["dense_solve" if case.get("zipf") == 0.0 else kind], 0
    if kind.startswith("sparse"):
        # a column index per nonzero and orientation, the value where the row's entries have one of their own, the vectors
        nnz = _nonzeros(case)
        entry = 12.0 if case["values"] == "lognormal" else 4.0
        product = 2 * entry * nnz + 8 * (3 * n + 3 * d)
        moved = (funs + products) * product + diags * product / 2
        if kind == "sparse_train":
            moved += 24.0 * nnz   # the arrays in, the transposed copy out
        return {"bytes": moved, "flops": (funs + products) * 4 * nnz + diags * 3 * nnz}
    K = _problems(case) if kind.startswith("batch") else 1
    per_row_D = 8.0 if case["loss"] == LR else 0.125
    product = 8 * n * d + K * n * per_row_D
    return {"bytes": (funs + products + diags) * product, "flops": (funs + products + diags) * 4 * n * d * K}


def tolerance(case):
    """Measured against the same call with its sums in another order (other layouts, grids and drivers of the library).  Single
    evaluations differ by rounding, 2e-16 to 4e-16 (a plain order of summation over millions of rows: some 1e-14), and dense
    solves by no more.  A sparse solve multiplies the rounding by what its inner iterations amplify: with Zipf-distributed
    features up to 1.2e-9 in w over forty drawn problems (3e-8 in single entries)."""
    if case["kind"] in ("sparse_solve", "sparse_train") and case["zipf"] > 0.0:
        return {"rel": 5e-9, "max": 1e-7}
    return {"rel": 1e-13, "max": 1e-11}
