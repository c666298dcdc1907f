"""The work that users of this library have it do, as cases that can be timed.

Four kinds of call, each through the package's public entry points:

  spmv     y <- alpha A x + beta y in one storage format
  convert  a matrix from CSR to another format and back, with the exports
  solve    a Krylov solve (or a fixed number of iterations of one)
  batch    many small independent systems solved by one call

Matrices are the synthetic families of the benchmark and the tests (grid
stencils, convection-diffusion, banded, block-diagonal, uniform and lognormal
random rows), made on the GPU from the case's seed.
"""
import math

import torch

import paper_2011_08879_amd as gko

DEV = "cuda"
DTYPES = {"f64": torch.float64, "f32": torch.float32}

#: Entries of one matrix at most: the 27-point stencil on 128^3.
MOST_NNZ = 56_000_000


# --------------------------------------------------------------------------- cases
def _spmv(name, kind, dims, fmt, dtype="f64", alpha=1.0, beta=0.0, **family):
    nx, ny, nz = dims
    return dict(name=name, do="spmv", kind=kind, nx=nx, ny=ny, nz=nz, fmt=fmt, dtype=dtype, alpha=alpha, beta=beta, **family)


def _convert(name, kind, dims, fmt, dtype="f64", **family):
    nx, ny, nz = dims
    return dict(name=name, do="convert", kind=kind, nx=nx, ny=ny, nz=nz, fmt=fmt, dtype=dtype, **family)


def _solve(name, solver, kind, dims, fmt, tol=1e-12, maxit=20000, block=0, mixed=False, krylov=30):
    nx, ny, nz = dims
    return dict(name=name, do="solve", solver=solver, kind=kind, nx=nx, ny=ny, nz=nz, fmt=fmt, tol=tol, maxit=maxit,
                block=block, mixed=mixed, krylov=krylov)


def listed():
    return [
        # The smallest product: a small 2D problem in the format that it is assembled in, bound by the call itself.
        _spmv("spmv_coo_lap2d_64", "star", (64, 64, 1), "coo"),
        # The regular matrix of the benchmark's sweep in the default format, the largest product.
        _spmv("spmv_csr_box3d_128", "box", (128, 128, 128), "csr"),
        # The irregular matrix of the sweep in the load-balanced format.
        _spmv("spmv_merge_lognormal_1m", "lognormal", (1_000_000, 1, 1), "csr_merge", mean=16, sigma=1.56),
        # FP32 and an accumulating product, an odd row count: the step y <- alpha A x + beta y of an iterative method.
        _spmv("spmv_coo_banded_333k_f32", "banded", (333_331, 1, 1), "coo", "f32", alpha=1.5, beta=0.5, mean=24, width=64),
        # A damped residual y <- y / 2 - A x of an irregular matrix in the hybrid format (an ELL product and a COO tail).
        _spmv("spmv_hybrid_lognormal_250k", "lognormal", (250_001, 1, 1), "hybrid", alpha=-1.0, beta=0.5, mean=16, sigma=1.56),
        # What choosing a format costs: CSR to ELL and back, with the arrays read out both times.
        _convert("convert_ell_banded_500k", "banded", (500_009, 1, 1), "ell", mean=16, width=48),
        # The smallest solve: the 2D Laplacian to 1e-12 (4,096 rows, unpreconditioned CG).
        _solve("cg_lap2d_64", "cg", "star", (64, 64, 1), "csr"),
        # An ordinary solve: 3D Poisson with 110,592 rows, unpreconditioned CG.
        _solve("cg_lap3d_48", "cg", "star", (48, 48, 48), "sellp"),
        # Nonsymmetric, ordinary size, a ragged grid: 32 steps of BiCGSTAB on convection-diffusion.
        _solve("bicgstab_convdiff_211x307", "bicgstab", "convdiff", (211, 307, 1), "ell", maxit=32),
        # Two cycles of GMRES(30) on a convection-diffusion problem of 22,500 rows.
        _solve("gmres_convdiff_150", "gmres", "convdiff", (150, 150, 1), "csr", maxit=60),
        # The largest solve of the benchmark: 16.8M rows, block-Jacobi CG in mixed precision.
        _solve("pcg_mixed_lap3d_256", "cg", "star", (256, 256, 256), "ell", tol=4e-13, block=8, mixed=True),
        # Ten thousand small systems in one call.
        dict(name="batch_10000_f64", do="batch", nsys=10_000, lo=32, hi=1024, dtype="f64"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid_dims(rng, n, d):
    """Edges of a ragged d-dimensional grid of about n points."""
    e = n ** (1.0 / d)
    dims = [max(2, int(round(e * rng.uniform(0.8, 1.25)))) for _ in range(d)]
    return tuple(dims + [1] * (3 - d))


def _draw_matrix(rng, n_hi):
    """A matrix of the families above: (kind, dims, family) and the formats that suit it."""
    kind = rng.choice(("star2", "star3", "box3", "banded", "uniform", "blocks", "lognormal", "lognormal"))
    n = _log(rng, 1000, n_hi)
    if kind in ("star2", "star3", "box3"):
        d = int(kind[-1])
        return kind[:-1], _grid_dims(rng, min(n, MOST_NNZ // (27 if kind == "box3" else 7)), d), {}, True
    mean = rng.randint(4, 48)
    n = min(n, MOST_NNZ // 2 // (mean + 1)) | 1
    if kind == "lognormal":
        return kind, (n, 1, 1), {"mean": mean, "sigma": round(rng.uniform(0.5, 2.0), 3)}, False
    if kind == "banded":
        return kind, (n, 1, 1), {"mean": mean, "width": rng.randint(max(8, mean), 64)}, True
    return kind, (n, 1, 1), {"mean": mean}, True


def draw(rng):
    do = rng.choice(("spmv",) * 5 + ("convert",) * 2 + ("solve",) * 5 + ("batch",) * 2)
    if do == "batch":
        lo = rng.randint(8, 200)
        return dict(do="batch", nsys=_log(rng, 50, 10_000), lo=lo, hi=rng.randint(lo, 1024), dtype=rng.choice(("f64", "f64", "f32")))
    if do == "solve":
        solver = rng.choice(("cg", "cg", "cg", "cg", "fcg", "pipecg", "bicgstab", "bicgstab", "cgs", "gmres"))
        fmt = rng.choice(("csr", "csr", "ell", "sellp", "csr_merge", "coo", "hybrid"))
        d = rng.choice((2, 3))
        if solver == "cg" and rng.random() < 0.25:
            case = _solve("", "cg", "star", _grid_dims(rng, _log(rng, 8000, 2_000_000), 3), fmt, block=rng.choice((0, 4, 8)), mixed=True)
        elif solver in ("cg", "fcg", "pipecg"):
            block = 0 if rng.random() < 0.5 else rng.choice((2, 4, 8, 16))
            case = _solve("", solver, "star", _grid_dims(rng, _log(rng, 1000, 4_000_000), d), fmt, block=block, maxit=rng.randint(30, 120))
        elif solver == "gmres":
            case = _solve("", solver, rng.choice(("convdiff", "star")), _grid_dims(rng, _log(rng, 1000, 1_000_000), 2), fmt,
                          maxit=rng.randint(20, 75), krylov=rng.choice((10, 20, 30, 30, 50)))
        else:
            case = _solve("", solver, "convdiff", _grid_dims(rng, _log(rng, 1000, 2_000_000), 2), fmt,
                          maxit=rng.randint(12, 32 if solver == "bicgstab" else 20))
    else:
        kind, dims, family, regular = _draw_matrix(rng, 2_000_000 if do == "spmv" else 1_000_000)
        dtype = rng.choice(("f64", "f64", "f32"))
        if do == "spmv":
            fmt = rng.choice(("csr", "csr", "csr_merge", "coo", "hybrid") + (("ell", "sellp") if regular else ()))
            alpha, beta = rng.choice(((1.0, 0.0), (1.0, 0.0), (-1.0, 0.5), (1.5, 0.5)))
            case = _spmv("", kind, dims, fmt, dtype, alpha, beta, **family)
        else:
            fmt = rng.choice(("coo", "hybrid", "csr_merge") + (("ell", "ell", "sellp", "sellp") if regular else ()))
            case = _convert("", kind, dims, fmt, dtype, **family)
    del case["name"]
    return case


# --------------------------------------------------------------------------- matrices
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform(n, g, dtype=torch.float64):
    return torch.rand(n, generator=g, device=DEV, dtype=dtype) * 2 - 1


def _offsets(kind, nx, ny, nz):
    """(dx, dy, dz) of a stencil's points, by ascending column."""
    r = range(-1, 2)
    points = [(dx, dy, dz) for dz in r for dy in r for dx in r]
    points = [p for p in points if all(d == 0 or e > 1 for d, e in zip(p, (nx, ny, nz)))]
    return points if kind == "box" else [p for p in points if sum(map(abs, p)) <= 1]


def _stencil_value(kind, p, nx, ny, nz):
    d = sum(e > 1 for e in (nx, ny, nz))
    if p == (0, 0, 0):
        return 3.0 ** d - 1 if kind == "box" else 2.0 * d
    if kind == "convdiff" and p[0]:
        return -1.0 + 0.5 * p[0]
    return -1.0


def _stencil(kind, nx, ny, nz):
    n = nx * ny * nz
    i = torch.arange(n, device=DEV, dtype=torch.int32)
    x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
    points = _offsets(kind, nx, ny, nz)
    ok = torch.empty((n, len(points)), dtype=torch.bool, device=DEV)
    for k, (dx, dy, dz) in enumerate(points):
        ok[:, k] = (x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) & (z + dz >= 0) & (z + dz < nz)
    off = torch.tensor([dx + nx * (dy + ny * dz) for dx, dy, dz in points], device=DEV, dtype=torch.int32)
    val = torch.tensor([_stencil_value(kind, p, nx, ny, nz) for p in points], device=DEV, dtype=torch.float64)
    col = (i[:, None] + off)[ok]
    return _row_ptr(ok.sum(1)), col, val.expand(n, -1)[ok]


def _row_ptr(lens):
    rp = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens, 0, out=rp[1:])
    return rp.to(torch.int32)


def _rows(rp):
    lens = (rp[1:] - rp[:-1]).long()
    return torch.repeat_interleave(torch.arange(lens.numel(), device=DEV), lens)


def _random_rows(lens, m, g):
    """About lens[i] distinct uniform columns in row i (repeated draws fall together)."""
    row = torch.repeat_interleave(torch.arange(lens.numel(), device=DEV), lens)
    col = (torch.rand(row.numel(), generator=g, device=DEV, dtype=torch.float64) * m).long().clamp_(max=m - 1)
    key = torch.unique(row * m + col)
    return _row_ptr(torch.bincount(key // m, minlength=lens.numel())), (key % m).to(torch.int32)


def _matrix(case, seed):
    """CSR arrays (row offsets and columns int32, values float64) of a case's matrix:
    values from the seed, and the pattern too, except in conversions, whose results
    are arrays of the pattern's sizes."""
    kind, n, values = case["kind"], case["nx"], _gen(seed)
    g = _gen(seed + 2 if case["do"] != "convert" else n)
    if kind in ("star", "box", "convdiff"):
        rp, col, val = _stencil(kind, case["nx"], case["ny"], case["nz"])
        # the products and conversions take variable coefficients, the solves the plain operator
        return rp, col, val if case["do"] == "solve" else val * (1 + 0.1 * _uniform(col.numel(), values))
    mean = case["mean"]
    if kind == "lognormal":  # longest row 10,000, as in the benchmark
        s = case["sigma"]
        z = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
        lens = torch.exp(math.log(mean) - s * s / 2 + s * z).round().clamp(1, min(n, 10000)).long()
        lens[int(torch.argmax(lens))] = min(n, 10000)
        rp, col = _random_rows(lens, n, g)
    elif kind == "uniform":
        lens = torch.randint(max(1, mean // 2), mean + mean // 2 + 1, (n,), generator=g, device=DEV)
        rp, col = _random_rows(lens, n, g)
    elif kind == "banded":
        w = case["width"]
        off = torch.arange(-w, w + 1, device=DEV, dtype=torch.int32)
        c = torch.arange(n, device=DEV, dtype=torch.int32)[:, None] + off
        pick = torch.rand((n, 2 * w + 1), generator=g, device=DEV) < (mean - 1) / (2 * w)
        pick[:, w] = True
        pick &= (c >= 0) & (c < n)
        rp, col = _row_ptr(pick.sum(1)), c[pick]
    else:  # dense diagonal blocks of 1 .. 2 mean rows
        size = torch.randint(1, 2 * mean + 1, (n,), generator=g, device=DEV)
        end = torch.cumsum(size, 0)
        k = int((end < n).sum()) + 1
        size, end = size[:k].clone(), end[:k].clone()
        size[-1] -= end[-1] - n
        start = torch.cumsum(size, 0) - size
        lens = torch.repeat_interleave(size, size)
        rp = _row_ptr(lens)
        row = _rows(rp)
        at = torch.arange(row.numel(), device=DEV) - rp[:-1].long()[row]
        col = (torch.repeat_interleave(start, size)[row] + at).to(torch.int32)
    return rp, col, _uniform(col.numel(), values)


def _product(A, x):
    """A x in 64 bits."""
    rp, col, val = A
    return torch.zeros(rp.numel() - 1, dtype=torch.float64, device=DEV).index_add_(0, _rows(rp), val.double() * x.double()[col.long()])


def _apply(case, v):
    """A v of a stencil case in 64 bits, from shifted copies of the grid."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    u = v.reshape(nz, ny, nx)
    p = torch.zeros((nz + 2, ny + 2, nx + 2), dtype=v.dtype, device=v.device)
    p[1:-1, 1:-1, 1:-1] = u
    out = torch.zeros_like(u)
    for dx, dy, dz in _offsets(case["kind"], nx, ny, nz):
        out += _stencil_value(case["kind"], (dx, dy, dz), nx, ny, nz) * p[1 + dz:1 + dz + nz, 1 + dy:1 + dy + ny, 1 + dx:1 + dx + nx]
    return out.reshape(-1)


# --------------------------------------------------------------------------- batches
def _batch(case, seed):
    """Small SPD systems as the benchmark's: m ~ U{lo..hi} rows, a 3- or 5-point
    pattern (grid width ceil(sqrt(m))), diagonal shift U[0.1, 2], x* ~ U[-1, 1].
    Sizes from the case, shifts and right-hand sides from the seed."""
    nsys = case["nsys"]
    g = _gen(nsys)
    m = torch.randint(case["lo"], case["hi"] + 1, (nsys,), generator=g, device=DEV)
    five = torch.rand(nsys, generator=g, device=DEV) < 0.5
    g = _gen(seed)
    shift = torch.rand(nsys, generator=g, device=DEV, dtype=torch.float64) * 1.9 + 0.1
    ro = torch.zeros(nsys + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(m, 0, out=ro[1:])
    s = torch.repeat_interleave(torch.arange(nsys, device=DEV), m)
    i = torch.arange(s.numel(), device=DEV) - ro[s]
    w = torch.sqrt(m.double()).ceil().long()[s]
    ms, f = m[s], five[s]
    ok = torch.stack((f & (i >= w), i % w > 0, torch.ones_like(f), (i % w < w - 1) & (i + 1 < ms), f & (i + w < ms)), 1)
    col = torch.stack((i - w, i - 1, i, i + 1, i + w), 1)[ok]
    val = torch.full((s.numel(), 5), -1.0, dtype=torch.float64, device=DEV)
    val[:, 2] = torch.where(f, 4.0, 2.0) + shift[s]
    val = val[ok]
    if case["dtype"] == "f32":
        val = val.float()
    lens = ok.sum(1)
    rp = _row_ptr(lens).long()
    no = rp[ro]
    rows = torch.repeat_interleave(torch.arange(s.numel(), device=DEV), lens)
    xs = _uniform(s.numel(), g)
    b = torch.zeros_like(xs).index_add_(0, rows, val.double() * xs[col + ro[s[rows]]])
    # local offsets, m + 1 of each system
    lp = torch.zeros(s.numel() + nsys, dtype=torch.int64, device=DEV)
    lp[torch.arange(s.numel(), device=DEV) + s] = rp[:-1] - no[s]
    lp[ro[1:] + torch.arange(nsys, device=DEV)] = no[1:] - no[:-1]
    return ro, no, lp.to(torch.int32), col.to(torch.int32), val, b, xs


# --------------------------------------------------------------------------- the calls
def prepare(case, seed):
    if case["do"] == "batch":
        ro, no, lp, col, val, b, _ = _batch(case, seed)
        B = gko.Batch(ro, no, lp, col, val, dtype=val.dtype)
        # the setting that the library's tuning of a 10,000-system batch keeps on disk
        B.block, B.lds_mode = 256, "waves"
        return dict(do="batch", B=B, b=b, x=torch.empty_like(b))
    ctx = gko.Context()
    A = _matrix(case, seed)
    g, n = _gen(seed + 1), A[0].numel() - 1
    if case["do"] == "solve":
        M = gko.Matrix.from_csr(*A, ctx=ctx).convert(case["fmt"])
        ctx.set_solver_opts(precision=gko.PREC_MIXED_IR if case["mixed"] else gko.PREC_FP64,
                            precond=gko.PRECOND_BLOCK_JACOBI if case["block"] else gko.PRECOND_NONE,
                            block_size=case["block"] or 8, krylov_dim=case["krylov"])
        b = _apply(case, _uniform(n, g))
        return dict(do="solve", M=M, call=getattr(gko, case["solver"]), b=b, x=torch.empty_like(b), tol=case["tol"], maxit=case["maxit"])
    dt = DTYPES[case["dtype"]]
    M = gko.Matrix.from_csr(A[0], A[1], A[2].to(dt), ctx=ctx)
    if case["do"] == "convert":
        return dict(do="convert", M=M, fmt=case["fmt"])
    M.convert(case["fmt"])
    return dict(do="spmv", M=M, alpha=case["alpha"], beta=case["beta"], x=_uniform(n, g).to(dt), y=_uniform(n, g).to(dt))


def run(state):
    do = state["do"]
    if do == "spmv":
        return gko.spmv(state["M"], state["alpha"], state["x"], state["beta"], state["y"])
    if do == "convert":
        M, fmt = state["M"], state["fmt"]
        M.convert(fmt)
        if fmt == "sellp":
            stored = M.export_sellp()
        elif fmt == "csr_merge":
            stored = M.export_csr()
        else:
            stored = M.export_storage()
        return [stored, M.convert("csr").export_csr()]
    if do == "solve":
        state["x"].zero_()
        state["call"](state["M"], state["b"], state["x"], tol=state["tol"], maxit=state["maxit"])
        return state["x"]
    # x is what the systems are solved for; iteration counts and residuals are diagnostics
    state["B"].solve(state["b"], state["x"], tol=1e-12, maxit=1000)
    return state["x"]


# --------------------------------------------------------------------------- what a call cannot do without
def _expected_nnz(case):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["kind"] in ("star", "box", "convdiff"):
        return sum((nx - abs(dx)) * (ny - abs(dy)) * (nz - abs(dz)) for dx, dy, dz in _offsets(case["kind"], nx, ny, nz))
    if case["kind"] == "blocks":  # sizes uniform in 1..2 mean, each row as long as its block
        return int(nx * (4 * case["mean"] + 1) / 3)
    return nx * case["mean"]


def _entry_bytes(fmt, s):
    return s + (8 if fmt == "coo" else 4)


def _iterations(case):
    """Iterations of a solve: its cap, or for a solve to its tolerance what CG on
    a Poisson matrix takes, about 0.2 sqrt(kappa) log(2 / tol)."""
    if case["maxit"] < 20000:
        return case["maxit"]
    e = max(case["nx"], case["ny"], case["nz"]) + 1
    return 0.2 * (2 * e / math.pi) * math.log(2 / case["tol"])


def work(case):
    if case["do"] == "batch":
        rows = case["nsys"] * (case["lo"] + case["hi"]) / 2
        s = 8 if case["dtype"] == "f64" else 4
        return {"bytes": rows * (4 * (s + 4) + 4 + 16), "flops": rows * 40 * (2 * 4 + 10)}
    n, nnz = case["nx"] * case["ny"] * case["nz"], _expected_nnz(case)
    if case["do"] == "solve":
        # each iteration reads the matrix (or twice, for the methods with two products) and
        # updates x, r and p: each read and written once
        its, s = _iterations(case), 4 if case["mixed"] else 8
        products = 2 if case["solver"] in ("bicgstab", "cgs") else 1
        basis = case["krylov"] if case["solver"] == "gmres" else 0
        inverse = n * (case["block"] + 1) / 2 * s
        one = products * nnz * _entry_bytes(case["fmt"], s) + (6 + basis / 2) * n * s + inverse
        return {"bytes": its * one, "flops": its * (products * 2 * nnz + 10 * n + 4 * basis / 2 * n)}
    s = 8 if case["dtype"] == "f64" else 4
    if case["do"] == "convert":
        # read and write CSR and the other format once, and once more for each export
        other = nnz * _entry_bytes(case["fmt"], s)
        return {"bytes": 3 * (nnz * (s + 4) + 4 * n) + 3 * other, "flops": 0}
    return {"bytes": nnz * _entry_bytes(case["fmt"], s) + 2 * n * s + (n * s if case["beta"] else 0), "flops": 2 * nnz}


# --------------------------------------------------------------------------- plain 64-bit results
def exact(case, seed):
    if case["do"] == "batch":
        return _batch(case, seed)[-1]
    if case["do"] == "solve":
        n = case["nx"] * case["ny"] * case["nz"]
        xs = _uniform(n, _gen(seed + 1))
        return xs if case["maxit"] >= 20000 else _krylov(case, _apply(case, xs))
    A = _matrix(case, seed)
    if case["do"] == "convert":
        return None  # copies: integers and bytes, and values that equal their inputs
    dt, n, g = DTYPES[case["dtype"]], A[0].numel() - 1, _gen(seed + 1)
    x, y = _uniform(n, g).to(dt), _uniform(n, g).to(dt)
    return case["alpha"] * _product((A[0], A[1], A[2].to(dt)), x) + case["beta"] * y.double()


def _blocks_apply(case, bs):
    """v -> M^-1 v with the inverses of the diagonal blocks of bs rows."""
    rp, col, val = _stencil(case["kind"], case["nx"], case["ny"], case["nz"])
    n, row = rp.numel() - 1, _rows(rp)
    nb = -(-n // bs)
    inside = row // bs == col.long() // bs
    D = torch.eye(bs, dtype=torch.float64, device=DEV).repeat(nb, 1, 1)
    r, c = row[inside], col[inside].long()
    D[r // bs, r % bs, c % bs] = val[inside]
    inv = torch.linalg.inv(D)

    def apply(v):
        p = torch.zeros(nb * bs, dtype=v.dtype, device=v.device)
        p[:n] = v
        return (inv * p.reshape(nb, 1, bs)).sum(2).reshape(-1)[:n]

    return apply


def _krylov(case, b):
    """The textbook iterations in 64 bits from x = 0, stopped by the cap or the tolerance."""
    A = lambda v: _apply(case, v)  # noqa: E731
    stop, maxit = case["tol"] * float(b.norm()), case["maxit"]
    x, r = torch.zeros_like(b), b.clone()
    if case["solver"] in ("cg", "fcg", "pipecg"):  # one iterate in exact arithmetic
        M = _blocks_apply(case, case["block"]) if case["block"] else lambda v: v.clone()
        z = M(r)
        p, rho = z.clone(), r @ z
        for _ in range(maxit):
            q = A(p)
            alpha = rho / (p @ q)
            x += alpha * p
            r -= alpha * q
            if float(r.norm()) <= stop:
                break
            z = M(r)
            rho, old = r @ z, rho
            p = z + (rho / old) * p
    elif case["solver"] == "bicgstab":
        rh, p, rho = r.clone(), r.clone(), r @ r
        for _ in range(maxit):
            v = A(p)
            alpha = rho / (rh @ v)
            s = r - alpha * v
            if float(s.norm()) <= stop:
                x += alpha * p
                break
            t = A(s)
            omega = (t @ s) / (t @ t)
            x += alpha * p + omega * s
            r = s - omega * t
            if float(r.norm()) <= stop:
                break
            rho, old = rh @ r, rho
            p = r + (rho / old) * (alpha / omega) * (p - omega * v)
    elif case["solver"] == "cgs":
        rh, u, p, rho = r.clone(), r.clone(), r.clone(), r @ r
        for _ in range(maxit):
            t = A(p)
            alpha = rho / (t @ rh)
            q = u - alpha * t
            x += alpha * (u + q)
            r = r - alpha * A(u + q)
            if float(r.norm()) <= stop:
                break
            rho, old = r @ rh, rho
            beta = rho / old
            u = r + beta * q
            p = u + beta * (q + beta * p)
    else:  # restarted GMRES: least squares over each cycle's Krylov basis
        left = maxit
        while left > 0 and float(r.norm()) > stop:
            k = min(case["krylov"], left)
            V, H = torch.zeros((k + 1, b.numel()), dtype=b.dtype, device=b.device), torch.zeros((k + 1, k), dtype=b.dtype)
            beta = float(r.norm())
            V[0] = r / beta
            for j in range(k):
                w = A(V[j])
                for _ in range(2):
                    h = V[: j + 1] @ w
                    w = w - h @ V[: j + 1]
                    H[: j + 1, j] += h.cpu()
                H[j + 1, j] = w.norm().cpu()
                V[j + 1] = w / w.norm()
            e = torch.zeros((k + 1, 1), dtype=b.dtype)
            e[0] = beta
            x = x + torch.linalg.lstsq(H, e).solution[:, 0].to(b.device) @ V[:k]
            r = b - A(x)
            left -= k
    return x
