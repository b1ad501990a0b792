"""The work that users of this library have it do, as timed cases.

A case is a dict of plain values; `prepare` makes what a program holds before
the call (device or host matrices, a batch plan, a workspace), `run` is one
pass through the public entry points, `work` counts the bytes and operations
the pass cannot do without, `exact` is the result in 64 bits.

Matrices are column-major in 1-D storage with leading dimensions, as
everywhere in the library.  Updates with beta != 0 work in place on C, so a
repeated pass continues from the C of the one before.
"""
import math

import numpy as np
import torch

import paper_1608_05265_amd as mg

SQUARE_SWEEP = dict(alpha=1.5, beta=-0.5, pad=16)


def _sgemm(name, ta, tb, m, n, k, mode="fp32", alpha=1.0, beta=0.0, pad=0, workspace=False):
    return {"name": name, "kind": "sgemm", "ta": ta, "tb": tb, "m": m, "n": n, "k": k, "mode": mode,
            "alpha": alpha, "beta": beta, "pad": pad, "workspace": workspace}


def listed():
    return [
        # the smallest ordinary call: one launch, bound by latency
        _sgemm("sgemm_256", "N", "N", 256, 256, 256),
        # sizes as an application's own dimensions come: odd, tight leading
        # dimensions, a transposed operand, an update of C
        _sgemm("sgemm_odd", "T", "N", 1511, 777, 1003, alpha=1.5, beta=-0.5),
        # the square sweep's smallest and largest sizes
        _sgemm("sgemm_1024", "N", "T", 1024, 1024, 1024, **SQUARE_SWEEP),
        _sgemm("sgemm_8192", "T", "N", 8192, 8192, 8192, **SQUARE_SWEEP),
        # trailing update of a blocked factorization: a stream over a large C
        _sgemm("sgemm_rank256", "N", "N", 16384, 16384, 256, alpha=-1.0, beta=1.0),
        # few outputs, long inner products
        _sgemm("sgemm_skinny", "N", "N", 128, 512, 8192, alpha=1.5, beta=-0.5),
        # the split-precision form with a workspace that the caller keeps
        _sgemm("sgemm_x3_4096", "N", "T", 4096, 4096, 4096, mode="bf16x3", workspace=True,
               **SQUARE_SWEEP),
        # many independent problems of mixed sizes in one planned launch
        {"name": "batch_512", "kind": "batch", "count": 512, "lo": 2, "hi": 64, "step": 16,
         "mode": "fp32"},
        # double precision on the FP64 matrix cores
        {"name": "dgemm_2048", "kind": "dgemm", "ta": "N", "tb": "N", "m": 2048, "n": 2048,
         "k": 2048, "alpha": 1.5, "beta": -0.5, "pad": 16},
        # Linpack: factor and solve, at the paper's N and at a large one
        {"name": "lu_4608", "kind": "lu", "n": 4608, "nrhs": 1, "mode": "fp32"},
        {"name": "lu_16384", "kind": "lu", "n": 16384, "nrhs": 1, "mode": "bf16x3"},
        # an unmodified BLAS caller, matrices in pageable host memory
        {"name": "host_4096", "kind": "host", "ta": "N", "tb": "N", "m": 4096, "n": 4096, "k": 4096,
         "alpha": 1.5, "beta": -0.5, "pad": 0},
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi]: half of them as they
    come, half rounded to a multiple of 16."""
    s = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if s >= 32 and rng.random() < 0.5:
        s = s // 16 * 16
    return max(lo, min(hi, s))


def draw(rng):
    kind = rng.choice(["sgemm", "sgemm", "sgemm", "rank", "skinny", "batch", "dgemm", "lu", "lu", "host"])
    ta, tb = rng.choice("NT"), rng.choice("NT")
    alpha, beta = rng.choice([(1.0, 0.0), (1.5, -0.5)])
    pad = rng.choice([0, 0, 16, 3])
    mode = rng.choice(["fp32", "fp32", "bf16x3"])
    if kind == "sgemm":  # any shape, up to 2 * 4096^3 operations
        m, n = _size(rng, 64, 6144), _size(rng, 64, 6144)
        k = _size(rng, 64, max(64, min(6144, 4096 ** 3 // (m * n))))
        c = _sgemm("", ta, tb, m, n, k, mode, alpha, beta, pad, mode == "bf16x3" and rng.random() < 0.5)
        del c["name"]
        return c
    if kind == "rank":  # rank-k updates of a large C
        c = _sgemm("", "N", "N", _size(rng, 4096, 16384), _size(rng, 4096, 16384), _size(rng, 64, 512),
                   mode, -1.0, 1.0, rng.choice([0, 16]))
        del c["name"]
        return c
    if kind == "skinny":
        c = _sgemm("", ta, tb, _size(rng, 32, 512), _size(rng, 32, 512), _size(rng, 2048, 16384), mode,
                   alpha, beta, pad)
        del c["name"]
        return c
    if kind == "batch":
        step = rng.choice([16, 16, 1])
        return {"kind": "batch", "count": _size(rng, 32, 512), "lo": 2 if step == 16 else 24,
                "hi": rng.randint(16, 64) if step == 16 else rng.randint(200, 700), "step": step,
                "mode": mode}
    if kind == "dgemm":
        return {"kind": "dgemm", "ta": ta, "tb": tb, "m": _size(rng, 64, 4096), "n": _size(rng, 64, 4096),
                "k": _size(rng, 64, 4096), "alpha": alpha, "beta": beta, "pad": pad}
    if kind == "lu":
        return {"kind": "lu", "n": _size(rng, 128, 8192), "nrhs": rng.choice([1, 1, 4, 32]), "mode": mode}
    return {"kind": "host", "ta": ta, "tb": tb, "m": _size(rng, 128, 4096), "n": _size(rng, 128, 4096),
            "k": _size(rng, 128, 4096), "alpha": alpha, "beta": beta, "pad": pad}


def _uniform(gen, count, dtype):
    x = torch.empty(count, dtype=dtype, device=gen.device)
    return x.uniform_(-1.0, 1.0, generator=gen)


def _matrices(case, seed, dtype, device):
    """A, B, C and their leading dimensions, all entries uniform in [-1, 1]
    (padding rows too)."""
    gen = torch.Generator(device=device).manual_seed(int(seed))
    m, n, k, pad = case["m"], case["n"], case["k"], case["pad"]
    ar, ac = (m, k) if case["ta"] == "N" else (k, m)
    br, bc = (k, n) if case["tb"] == "N" else (n, k)
    lda, ldb, ldc = ar + pad, br + pad, m + pad
    A, B = _uniform(gen, lda * ac, dtype), _uniform(gen, ldb * bc, dtype)
    return A, lda, B, ldb, _uniform(gen, ldc * n, dtype), ldc


def _batch_specs(case):
    """Sizes step * U{lo..hi}, transposes uniform over NN/NT/TN, beta over
    {0, 1}: the mix is the case's, the values the seed's."""
    rng = np.random.default_rng(160805265 + case["count"] * 1000 + case["hi"])
    out = []
    for _ in range(case["count"]):
        m, n, k = (int(case["step"] * v) for v in rng.integers(case["lo"], case["hi"] + 1, size=3))
        ta, tb = [("N", "N"), ("N", "T"), ("T", "N")][int(rng.integers(0, 3))]
        out.append((ta, tb, m, n, k, float(rng.integers(0, 2))))
    return out


def _batch_matrices(case, seed):
    specs = _batch_specs(case)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    A = _uniform(gen, sum(m * k for _, _, m, _, k, _ in specs), torch.float32)
    B = _uniform(gen, sum(k * n for _, _, _, n, k, _ in specs), torch.float32)
    C = _uniform(gen, sum(m * n for _, _, m, n, _, _ in specs), torch.float32)
    views, a, b, c = [], 0, 0, 0
    for ta, tb, m, n, k, beta in specs:
        views.append((ta, tb, m, n, k, beta, A[a:a + m * k], B[b:b + k * n], C[c:c + m * n]))
        a, b, c = a + m * k, b + k * n, c + m * n
    return views, C


def _system(case, seed):
    """A well-conditioned system with its rows in random order: uniform
    entries, and in each column one entry of 2 sqrt(n) on top, which is the
    column's pivot.  (The factors of a matrix of uniform entries alone hinge
    on the last bit of every entry and its solution has few correct digits
    in single precision.)"""
    n = case["n"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    A = _uniform(gen, n * n, torch.float32)
    perm = torch.randperm(n, generator=gen, device="cuda")
    A[torch.arange(n, device="cuda") * n + perm] += 2.0 * math.sqrt(n)
    return A, _uniform(gen, n * case["nrhs"], torch.float32)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "sgemm":
        s["A"], s["lda"], s["B"], s["ldb"], s["C"], s["ldc"] = _matrices(case, seed, torch.float32, "cuda")
        s["mode"] = mg.MODES[case["mode"]]
        if case["workspace"]:
            s["bytes"] = mg.workspace_size(case["ta"], case["tb"], case["m"], case["n"], case["k"], s["mode"])
            s["ws"] = torch.empty(s["bytes"] // 4 + 4, dtype=torch.float32, device="cuda")
    elif kind == "batch":
        views, s["C"] = _batch_matrices(case, seed)
        problems = [(ta, tb, m, n, k, 1.0, A, m if ta == "N" else k, B, k if tb == "N" else n, beta, C, m)
                    for ta, tb, m, n, k, beta, A, B, C in views]
        s["plan"] = mg.Batch(problems, mode=mg.MODES[case["mode"]])
    elif kind == "dgemm":
        s["A"], s["lda"], s["B"], s["ldb"], s["C"], s["ldc"] = _matrices(case, seed, torch.float64, "cuda")
    elif kind == "lu":
        # the matrix and right-hand sides are kept for the residual, the
        # factors and the solution have their own storage
        s["A"], s["b"] = _system(case, seed)
        s["LU"], s["x"] = torch.empty_like(s["A"]), torch.empty_like(s["b"])
        s["ipiv"] = torch.empty(case["n"], dtype=torch.int64, device="cuda")
        s["info"] = torch.empty(1, dtype=torch.int32, device="cuda")
        s["mode"] = mg.MODES[case["mode"]]
    else:
        A, s["lda"], B, s["ldb"], C, s["ldc"] = _matrices(case, seed, torch.float32, "cpu")
        s["A"], s["B"], s["C"] = A.numpy(), B.numpy(), C.numpy()
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "sgemm":
        if c["workspace"]:
            mg.sgemm_ws(c["ta"], c["tb"], c["m"], c["n"], c["k"], c["alpha"], s["A"], s["lda"], s["B"], s["ldb"],
                        c["beta"], s["C"], s["ldc"], s["mode"], s["ws"], s["bytes"])
        else:
            mg.sgemm(c["ta"], c["tb"], c["m"], c["n"], c["k"], c["alpha"], s["A"], s["lda"], s["B"], s["ldb"],
                     c["beta"], s["C"], s["ldc"], mode=s["mode"])
        return s["C"]
    if kind == "batch":
        s["plan"].launch()
        return s["C"]
    if kind == "dgemm":
        mg.dgemm(c["ta"], c["tb"], c["m"], c["n"], c["k"], c["alpha"], s["A"], s["lda"], s["B"], s["ldb"],
                 c["beta"], s["C"], s["ldc"])
        return s["C"]
    if kind == "lu":
        n = c["n"]
        s["LU"].copy_(s["A"])
        s["x"].copy_(s["b"])
        mg.sgetrf(n, s["LU"], n, s["ipiv"], s["info"], mode=s["mode"])
        mg.sgetrs(n, c["nrhs"], s["LU"], n, s["ipiv"], s["x"], n, mode=s["mode"])
        return {"LU": s["LU"], "ipiv": s["ipiv"], "info": s["info"], "x": s["x"]}
    mg.sgemm_host(c["ta"], c["tb"], c["m"], c["n"], c["k"], c["alpha"], s["A"], s["lda"], s["B"], s["ldb"],
                  c["beta"], s["C"], s["ldc"])
    return s["C"]


def work(case):
    kind = case["kind"]
    if kind == "batch":
        specs = _batch_specs(case)
        return {"bytes": sum(4 * (m * k + k * n + (2 if beta else 1) * m * n) for _, _, m, n, k, beta in specs),
                "flops": sum(2 * m * n * k for _, _, m, n, k, _ in specs)}
    if kind == "lu":
        n, r = case["n"], case["nrhs"]
        return {"bytes": 8 * n * n + 8 * n + 8 * n * r, "flops": 2 * n ** 3 // 3 + 2 * n * n * r}
    m, n, k = case["m"], case["n"], case["k"]
    size = 8 if kind == "dgemm" else 4
    return {"bytes": size * (m * k + k * n + (2 if case["beta"] else 1) * m * n), "flops": 2 * m * n * k}


def _product(ta, tb, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc):
    """C after the update, in 64 bits, in C's own layout."""
    a, b, c = A.double().view(-1, lda), B.double().view(-1, ldb), C.double().view(n, ldc).clone()
    # a stored column-major matrix is the transpose of its row-major view
    op_a = a[:, :m].T if ta == "N" else a[:, :k]
    op_b = b[:, :k].T if tb == "N" else b[:, :n]
    r = alpha * (op_a @ op_b).T
    c[:, :m] = r + beta * c[:, :m] if beta else r
    return c.view(-1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        views, C = _batch_matrices(case, seed)
        return torch.cat([_product(ta, tb, m, n, k, 1.0, A, m if ta == "N" else k, B, k if tb == "N" else n,
                                   beta, c, m) for ta, tb, m, n, k, beta, A, B, c in views])
    if kind == "dgemm":
        # the library's kernels and this sum in 64 bits differ by rounding alone
        A, lda, B, ldb, C, ldc = _matrices(case, seed, torch.float64, "cuda")
        return _product(case["ta"], case["tb"], case["m"], case["n"], case["k"], case["alpha"], A, lda, B, ldb,
                        case["beta"], C, ldc)
    if kind == "lu":
        n = case["n"]
        if n > 5000:  # the 64-bit factorization on the host takes too long
            return None
        A, b = _system(case, seed)
        a = A.view(n, n).T.double().cpu()
        lu, piv = torch.linalg.lu_factor(a)
        x = torch.linalg.lu_solve(lu, piv, b.view(-1, n).T.double().cpu())
        return {"LU": lu.T.contiguous().view(-1), "ipiv": None, "info": None, "x": x.T.contiguous().view(-1)}
    A, lda, B, ldb, C, ldc = _matrices(case, seed, torch.float32, "cuda" if kind == "sgemm" else "cpu")
    if kind == "host":
        A, B, C = A.cuda(), B.cuda(), C.cuda()
    out = _product(case["ta"], case["tb"], case["m"], case["n"], case["k"], case["alpha"], A, lda, B, ldb,
                   case["beta"], C, ldc)
    return out.cpu().numpy() if kind == "host" else out
