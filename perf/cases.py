"""Performance cases of the SpGEMM library, each through a public entry point.

Every input is made on the GPU.  A case's pattern is drawn once from its sizes
(so that nnz(C) is the same for every seed); the seed draws the values and,
where the pattern has no order of its own (all but bands and grids), the
permutation of the rows, of the inner index and of the columns.  The sizes are
those of the repository's own workloads (``synthetic/gen.py``) or the same
shapes at smaller, ragged sizes.  Kinds:

  square    C = A*A, uniform or power-law rows             (``spgemm``)
  galerkin  the two products of an algebraic-multigrid     (``spgemm`` twice)
            set-up, R*(A*P) or (R*A)*P
  narrow    A tall and square, B with few columns, pattern (``Plan.compute``)
            analysed once and multiplied with new values
  once      many independent products of uneven sizes,     (``batch_multiply``)
            seen once
  replay    the same kind, recomputed on fixed patterns    (``Batch.run``)
  train     forward and backward of 0.5*|A*B|^2 through    (``matmul``)
            autograd
  step      forward and backward on an analysed pattern    (``Plan.compute``,
                                                            ``Plan.backward``)
"""
import math
import zlib

import numpy as np
import torch

from paper_1504_05022_amd import Batch, CsrMatrix, Plan, batch_multiply, matmul, spgemm

DEV = "cuda"
DTYPES = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # the smallest call: a block of a larger method, launches and read-backs only
        {"name": "tiny_square_f32", "kind": "square", "dtype": "f32", "n": 317, "mean": 5.0,
         "gamma": 0.0, "cap": 5},
        # workload 1: a small uniform product, still bound by latency
        {"name": "uniform_square_f64", "kind": "square", "dtype": "f64", "n": 2000, "mean": 10.0,
         "gamma": 0.0, "cap": 10},
        # workload 2, the headline: a graph-like matrix squared, few rows hold most products
        {"name": "powerlaw_square_f64", "kind": "square", "dtype": "f64", "n": 200000,
         "mean": 16.0, "gamma": 2.1, "cap": 20000},
        # the same use at a ragged size in single precision, short rows dominate
        {"name": "powerlaw_square_f32", "kind": "square", "dtype": "f32", "n": 77777,
         "mean": 9.0, "gamma": 2.3, "cap": 3001},
        # workload 3: the set-up of a multigrid level, 27-point operator on 64^3
        {"name": "galerkin_27pt_f64", "kind": "galerkin", "dtype": "f64", "dim": 3, "points": 27,
         "g": 64, "order": "R(AP)"},
        # the multigrid experiment's 9-point operator, other order, odd grid
        {"name": "galerkin_9pt_f64", "kind": "galerkin", "dtype": "f64", "dim": 2, "points": 9,
         "g": 1023, "order": "(RA)P"},
        # a product with a narrow matrix whose pattern is kept: every long row is one dense window
        {"name": "narrow_compute_f64", "kind": "narrow", "dtype": "f64", "n": 90001, "mean": 18.0,
         "gamma": 2.2, "cap": 90001, "cols": 2000, "bdeg": 24},
        # workload 4 as it arrives: uneven banded problems, both precisions, seen once
        {"name": "batch_once_mixed", "kind": "once", "count": 20, "nmin": 1024, "nmax": 65536,
         "dmin": 4, "dmax": 32, "band": 0.05},
        # workload 4 with fixed patterns, replayed
        {"name": "batch_replay_mixed", "kind": "replay", "count": 20, "nmin": 1024,
         "nmax": 32768, "dmin": 4, "dmax": 32, "band": 0.05},
        # workload 5: a training step through autograd, narrow right operand
        {"name": "train_narrow_f32", "kind": "train", "dtype": "f32", "n": 300000, "mean": 20.0,
         "gamma": 2.2, "cap": 300000, "cols": 4096, "bdeg": 32},
        # a step on an analysed pattern, wide right operand
        {"name": "step_wide_f64", "kind": "step", "dtype": "f64", "n": 50000, "mean": 12.0,
         "gamma": 2.2, "cap": 5000, "cols": 50000, "bdeg": 12},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["square", "square", "galerkin", "narrow", "once", "replay", "train",
                       "step"])
    dt = rng.choice(["f32", "f64"])
    if kind == "square":
        n = _log_int(rng, 300, 150000)
        if rng.random() < 0.5:
            d = rng.randint(2, 14)
            return {"kind": kind, "dtype": dt, "n": n, "mean": float(d), "gamma": 0.0, "cap": d}
        return {"kind": kind, "dtype": dt, "n": n, "mean": rng.uniform(4.0, 14.0),
                "gamma": rng.uniform(2.1, 2.6), "cap": max(20, n // rng.randint(10, 40))}
    if kind == "galerkin":
        dim = rng.choice([2, 3])
        g = rng.randint(100, 1000) if dim == 2 else rng.randint(16, 63)
        points = rng.choice([2 * dim + 1, 3 ** dim])
        return {"kind": kind, "dtype": dt, "dim": dim, "points": points, "g": g,
                "order": rng.choice(["R(AP)", "(RA)P"])}
    if kind in ("once", "replay"):
        return {"kind": kind, "count": rng.randint(4, 20), "nmin": rng.randint(300, 1500),
                "nmax": _log_int(rng, 3000, 30000), "dmin": rng.randint(1, 8),
                "dmax": rng.randint(16, 32), "band": rng.uniform(0.02, 0.2)}
    if kind in ("narrow", "train"):
        n = _log_int(rng, 3000, 200000)
        return {"kind": kind, "dtype": dt, "n": n, "mean": rng.uniform(5.0, 20.0),
                "gamma": rng.uniform(2.15, 2.6), "cap": n,
                "cols": _log_int(rng, 100, 2048 if dt == "f64" else 4096),
                "bdeg": rng.randint(4, 32)}
    n = _log_int(rng, 3000, 50000)
    return {"kind": kind, "dtype": dt, "n": n, "mean": rng.uniform(4.0, 12.0),
            "gamma": rng.uniform(2.15, 2.6), "cap": max(20, n // 10),
            "cols": _log_int(rng, 5000, 60000), "bdeg": rng.randint(4, 14)}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _xmin(gamma, mean, cap):
    """Lower end of the truncated power law x^-gamma on [x_min, cap] with this mean."""
    def mean_of(x):
        a, b = 1.0 - gamma, 2.0 - gamma
        return (cap ** b - x ** b) / b / ((cap ** a - x ** a) / a)
    lo, hi = 0.5, float(mean)
    for _ in range(80):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if mean_of(mid) < mean else (lo, mid)
    return hi


def _pareto(u, gamma, mean, cap):
    e = 1.0 - gamma
    a, b = _xmin(gamma, mean, cap) ** e, float(cap) ** e
    return (a - u * (a - b)) ** (1.0 / e)


def _degrees(g, n, mean, gamma, cap):
    if gamma == 0.0:
        return torch.full((n,), int(cap), dtype=torch.int64, device=DEV)
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    return _pareto(u, gamma, mean, cap).round().long().clamp(1, int(cap))


def _csr(pg, g, rows, cols, deg, dtype, lo=None, width=None, perm=None):
    """Rows of distinct columns drawn uniformly by ``pg`` (a column drawn
    twice counts once), of [0, cols) or of a window per row, then permuted by
    ``perm`` (rows, columns); normal values drawn by ``g``."""
    r = torch.repeat_interleave(torch.arange(rows, device=DEV), deg.clamp(max=cols))
    x = torch.rand(r.numel(), generator=pg, device=DEV, dtype=torch.float64)
    c = (x * (cols if width is None else width)).long()
    if lo is not None:
        c = c + lo[r]
    key = torch.unique(r * cols + c)
    r = key // cols
    if perm is not None:
        key = torch.sort(perm[0][r] * cols + perm[1][key - r * cols])[0]
        r = key // cols
    rp = torch.zeros(rows + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(r, minlength=rows), 0)
    v = torch.randn(key.numel(), generator=g, device=DEV, dtype=torch.float64).to(dtype)
    return CsrMatrix((rows, cols), rp, (key - r * cols).int(), v)


def _stencil(g, n, dim, points, dtype):
    """Variable-coefficient stencil of the n^dim grid, truncated at the
    boundary: off-diagonals -U[0.5, 1.5], diagonal points - 1."""
    size = n ** dim
    f = torch.arange(size, device=DEV)
    coord = [(f // n ** k) % n for k in range(dim)]
    keys = []
    for o in range(3 ** dim):
        off = [(o // 3 ** k) % 3 - 1 for k in range(dim)]
        if points == 2 * dim + 1 and sum(abs(x) for x in off) > 1:
            continue
        ok = torch.ones(size, dtype=torch.bool, device=DEV)
        for k in range(dim):
            ok &= (coord[k] + off[k] >= 0) & (coord[k] + off[k] < n)
        r = f[ok]
        keys.append(r * size + r + sum(off[k] * n ** k for k in range(dim)))
    key = torch.sort(torch.cat(keys))[0]
    r = key // size
    c = key - r * size
    rp = torch.zeros(size + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(r, minlength=size), 0)
    v = -0.5 - torch.rand(key.numel(), generator=g, device=DEV, dtype=torch.float64)
    v = torch.where(r == c, torch.full_like(v, float(points - 1)), v)
    return CsrMatrix((size, size), rp, c.int(), v.to(dtype))


def _transfer(n, dim, dtype):
    """Prolongation of unsmoothed aggregation (blocks of two points per side)
    and its transpose."""
    h = (n + 1) // 2
    f = torch.arange(n ** dim, device=DEV)
    agg = sum(((f // n ** k) % n // 2) * h ** k for k in range(dim))
    one = torch.ones(f.numel(), dtype=dtype, device=DEV)
    nc = h ** dim
    P = CsrMatrix((f.numel(), nc), torch.arange(f.numel() + 1, device=DEV).int(), agg.int(), one)
    rp = torch.zeros(nc + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(agg, minlength=nc), 0)
    R = CsrMatrix((nc, f.numel()), rp, torch.sort(agg, stable=True)[1].int(), one.clone())
    return P, R


def _sizes(case):
    """Sizes of a batch: log-uniform, at fixed places of the range."""
    k = case["count"]
    a, b = math.log(case["nmin"]), math.log(case["nmax"])
    return [int(round(math.exp(a + (b - a) * (p + 0.5) / k))) for p in range(k)]


def _matrices(case, seed):
    sizes = sorted((k, v) for k, v in case.items() if k != "name")
    pg, g = _gen(zlib.crc32(repr(sizes).encode())), _gen(seed)
    kind = case["kind"]
    if kind in ("once", "replay"):
        pairs = []
        for p, n in enumerate(_sizes(case)):
            dt = torch.float64 if p % 2 == 0 else torch.float32
            w = max(case["dmax"], int(math.ceil(case["band"] * n)))
            lo = (torch.arange(n, device=DEV) - w // 2).clamp(0, n - w)
            pairs.append(tuple(
                _csr(pg, g, n, n, torch.randint(case["dmin"], case["dmax"] + 1, (n,),
                                                generator=pg, device=DEV), dt, lo, w)
                for _ in range(2)))
        return pairs
    dt = DTYPES[case["dtype"]]
    if kind == "galerkin":
        A = _stencil(g, case["g"], case["dim"], case["points"], dt)
        return (A,) + _transfer(case["g"], case["dim"], dt)
    n = case["n"]

    def shuffled(size):
        return torch.randperm(size, generator=g, device=DEV)

    inner = shuffled(n)
    rows = inner if kind == "square" else shuffled(n)
    A = _csr(pg, g, n, n, _degrees(pg, n, case["mean"], case["gamma"], case["cap"]), dt,
             perm=(rows, inner))
    if kind == "square":
        return A, A
    B = _csr(pg, g, n, case["cols"], torch.full((n,), case["bdeg"], device=DEV), dt,
             perm=(inner, shuffled(case["cols"])))
    return A, B


def prepare(case, seed):
    mats = _matrices(case, seed)
    kind = case["kind"]
    state = {"kind": kind, "mats": mats, "order": case.get("order")}
    if kind in ("narrow", "step"):
        state["plan"] = Plan(*mats)
    elif kind == "replay":
        state["batch"] = Batch(mats)
    elif kind == "train":
        for M in mats:
            M.val.requires_grad_(True)
    return state


# -------------------------------------------------------------------- passes

def _arrays(C):
    return [C.row_ptr, C.col_idx, C.val]


def run(state):
    kind, mats = state["kind"], state["mats"]
    if kind == "square":
        return _arrays(spgemm(*mats))
    if kind == "galerkin":
        A, P, R = mats
        X = spgemm(A, P) if state["order"] == "R(AP)" else spgemm(R, A)
        C = spgemm(R, X) if state["order"] == "R(AP)" else spgemm(X, P)
        return _arrays(X) + _arrays(C)
    if kind == "narrow":
        return _arrays(state["plan"].compute())
    if kind == "once":
        return [_arrays(C) for C in batch_multiply(mats)]
    if kind == "replay":
        return [_arrays(C) for C in state["batch"].run()]
    if kind == "train":
        # the gradient of 0.5 * |C|^2 with respect to C's values is C's values
        C = matmul(*mats)
        grads = torch.autograd.grad(C.val, [M.val for M in mats], C.val.detach())
        return [C.row_ptr, C.col_idx, C.val.detach()] + list(grads)
    C = state["plan"].compute()
    return _arrays(C) + list(state["plan"].backward(C, C.val))


# ----------------------------------------------------------------- reference

def _expand(A, B):
    """Every product of A*B: its entry of A, its entry of B, its key in C."""
    acol, brp = A.col_idx.long(), B.row_ptr.long()
    length = brp[acol + 1] - brp[acol]
    first = torch.cumsum(length, 0) - length
    e = torch.repeat_interleave(torch.arange(acol.numel(), device=DEV), length)
    b = brp[acol[e]] + torch.arange(e.numel(), device=DEV) - first[e]
    arp = A.row_ptr.long()
    row = torch.repeat_interleave(torch.arange(A.shape[0], device=DEV), arp[1:] - arp[:-1])
    return e, b, row[e] * B.shape[1] + B.col_idx[b].long()


def _product(A, B, grad=False):
    e, b, key = _expand(A, B)
    uniq, at = torch.unique(key, return_inverse=True)
    del key
    av, bv = A.val.detach().double(), B.val.detach().double()
    val = torch.zeros(uniq.numel(), dtype=torch.float64, device=DEV)
    val.index_add_(0, at, av[e] * bv[b])
    rows = uniq // B.shape[1]
    rp = torch.zeros(A.shape[0] + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=A.shape[0]), 0)
    C = CsrMatrix((A.shape[0], B.shape[1]), rp, (uniq - rows * B.shape[1]).int(), val)
    if not grad:
        return C
    y = val[at]
    dA = torch.zeros_like(av).index_add_(0, e, y * bv[b])
    dB = torch.zeros_like(bv).index_add_(0, b, y * av[e])
    return C, dA, dB


def exact(case, seed):
    mats = _matrices(case, seed)
    kind = case["kind"]
    if kind in ("once", "replay"):
        return [_arrays(_product(A, B)) for A, B in mats]
    if kind == "galerkin":
        A, P, R = mats
        X = _product(A, P) if case["order"] == "R(AP)" else _product(R, A)
        C = _product(R, X) if case["order"] == "R(AP)" else _product(X, P)
        return _arrays(X) + _arrays(C)
    if kind in ("train", "step"):
        C, dA, dB = _product(*mats, grad=True)
        return _arrays(C) + [dA, dB]
    return _arrays(_product(*mats))


# ---------------------------------------------------------------------- work

def _csr_bytes(rows, nnz, vb):
    return 4.0 * (rows + 1) + nnz * (4 + vb)


def _filled(u, width):
    """Expected distinct columns of u uniform products in `width` columns."""
    return width * -np.expm1(-np.asarray(u, dtype=np.float64) / width)


def _expected(case):
    """(nnz(A), products, nnz(C)) of a product of drawn rows, by expectation."""
    n = case["n"]
    if case["gamma"] == 0.0:
        d = np.array([float(case["cap"])])
    else:
        q = (np.arange(8192) + 0.5) / 8192
        d = np.clip(np.rint(_pareto(q, case["gamma"], case["mean"], case["cap"])), 1,
                    case["cap"])
    d = _filled(d, n)
    cols = n if case["kind"] == "square" else case["cols"]
    bd = float(d.mean()) if case["kind"] == "square" else float(_filled(case["bdeg"], cols))
    return n * float(d.mean()), n * float(d.mean()) * bd, n * float(_filled(d * bd, cols).mean())


def work(case):
    """Bytes: every input read once, every output written once."""
    kind = case["kind"]
    if kind in ("once", "replay"):
        total = flops = 0.0
        for p, n in enumerate(_sizes(case)):
            vb = 8 if p % 2 == 0 else 4
            w = max(case["dmax"], int(math.ceil(case["band"] * n)))
            d = float(_filled((case["dmin"] + case["dmax"]) / 2, w))
            c = float(_filled(d * d, min(n, 1.5 * w)))
            total += 2 * _csr_bytes(n, n * d, vb) + _csr_bytes(n, n * c, vb)
            flops += 2.0 * n * d * d
        return {"bytes": total, "flops": flops}
    vb = 4 if case["dtype"] == "f32" else 8
    if kind == "galerkin":
        g, dim, points = case["g"], case["dim"], case["points"]
        n, h = g ** dim, (g + 1) // 2
        nc = h ** dim
        box = points == 3 ** dim
        nnz = (3 * g - 2) ** dim if box else n * points - 2 * dim * g ** (dim - 1)
        coarse = (3 * h - 2) ** dim if box else nc * points - 2 * dim * h ** (dim - 1)
        left = 2 ** dim if box else dim + 1      # coarse neighbours of a fine row
        wide = 4 ** dim if box else 2 ** dim + 2 * dim * 2 ** (dim - 1)  # fine ones of a block
        mid_rows, mid = (n, n * left) if case["order"] == "R(AP)" else (nc, nc * wide)
        second = n * left if case["order"] == "R(AP)" else nc * wide
        total = (_csr_bytes(n, nnz, vb) + 2 * _csr_bytes(n, n, vb)
                 + 2 * _csr_bytes(mid_rows, mid, vb) + _csr_bytes(nc, coarse, vb))
        return {"bytes": total, "flops": 2.0 * nnz + 2.0 * second}
    nnz_a, products, nnz_c = _expected(case)
    n = case["n"]
    out = _csr_bytes(n, nnz_c, vb)
    if kind == "square":
        return {"bytes": _csr_bytes(n, nnz_a, vb) + out, "flops": 2 * products}
    nnz_b = products / max(nnz_a, 1.0) * n
    ins = _csr_bytes(n, nnz_a, vb) + _csr_bytes(n, nnz_b, vb)
    if kind == "narrow":
        return {"bytes": ins + out, "flops": 2 * products}
    # backward: A, B, C's pattern and its gradient read, both gradients written
    return {"bytes": 2 * (ins + out) + vb * (nnz_a + nnz_b), "flops": 6 * products}
