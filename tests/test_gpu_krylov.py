"""GPU parity of the Krylov solvers beyond CG and BiCGSTAB: flexible CG, CGS
and restarted GMRES, each against its pinned FP64 oracle on the same seeded
inputs (iteration counts within the rounding slack of the stopping tests,
true residuals, manufactured-solution error bounds), in several storage
formats, plus their status paths."""
import math

import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2011_08879_amd as g
    return g


@pytest.fixture()
def ctx(g):
    c = g.default_context()
    c.set_solver_opts()
    yield c
    c.set_solver_opts()


def relres(orc, A, b, x):
    return np.linalg.norm(b - orc.spmv(A, x)) / np.linalg.norm(b)


# --------------------------------------------------------------------------- FCG
@pytest.mark.parametrize("fmt", ["csr", "ell", "sellp", "coo"])
def test_fcg_laplace2d_matches_oracle(g, orc, gen_mod, ctx, fmt):
    N = 64
    A = gen_mod.laplace2d(N)
    xs = gen_mod.uniform(2, N * N)
    b = orc.spmv(A, xs)
    rc, xo, info_o = orc.fcg(A, b, tol=1e-10)
    M = g.Matrix.from_csr(*A).convert(fmt)
    x = dev(np.zeros(N * N))
    info = g.fcg(M, dev(b), x, tol=1e-10, maxit=5000)
    assert info["status"] == g.OK, info
    assert abs(info["iterations"] - info_o["iters"]) <= 2, (info, info_o)
    xg = host(x)
    assert relres(orc, A, b, xg) <= 1e-10
    kappa = (4 + 4 * math.cos(math.pi / (N + 1))) / (4 - 4 * math.cos(math.pi / (N + 1)))
    assert np.linalg.norm(xg - xo) / np.linalg.norm(xo) <= 2 * kappa * 1e-10


def test_fcg_block_jacobi_and_mixed(g, orc, gen_mod, ctx):
    N = 24
    A = gen_mod.laplace3d(N)
    n = N ** 3
    b = orc.spmv(A, gen_mod.uniform(5, n))
    rc, inv = orc.bj_invert(A, 8)
    rc, xo, info_o = orc.fcg(A, b, tol=1e-10, bj_inv=inv)
    M = g.Matrix.from_csr(*A)
    ctx.set_solver_opts(precond=g.PRECOND_BLOCK_JACOBI, block_size=8)
    x = dev(np.zeros(n))
    info = g.fcg(M, dev(b), x, tol=1e-10)
    assert info["status"] == g.OK and abs(info["iterations"] - info_o["iters"]) <= 2, (info, info_o)
    assert relres(orc, A, b, host(x)) <= 1e-10
    # with a fixed SPD preconditioner FCG and CG agree up to rounding
    xc = dev(np.zeros(n))
    infoc = g.cg(M, dev(b), xc, tol=1e-10)
    assert abs(infoc["iterations"] - info["iterations"]) <= 1
    ctx.set_solver_opts(precision=g.PREC_MIXED_IR, precond=g.PRECOND_BLOCK_JACOBI, block_size=8)
    x = dev(np.zeros(n))
    info = g.fcg(M, dev(b), x, tol=1e-10)
    assert info["status"] == g.OK and info["outer_iterations"] >= 2
    assert relres(orc, A, b, host(x)) <= 1e-10


def test_fcg_statuses(g, gen_mod, ctx):
    L = g.Matrix.from_csr(*gen_mod.laplace2d(32))
    info = g.fcg(L, dev(np.zeros(1024)), dev(np.ones(1024)))
    assert info["status"] == g.OK and info["iterations"] == 0
    info = g.fcg(L, dev(np.ones(1024)), dev(np.zeros(1024)), tol=1e-10, maxit=5)
    assert info["status"] == g.ERR_NOT_CONVERGED and info["iterations"] == 5
    D = g.Matrix.from_csr(np.arange(5, dtype=np.int32), np.arange(4, dtype=np.int32),
                          np.array([1.0, 2.0, -1.0, 3.0]))
    assert g.fcg(D, dev(np.ones(4)), dev(np.zeros(4)))["status"] == g.ERR_NOT_SPD


# --------------------------------------------------------------------------- CGS
@pytest.mark.parametrize("fmt", ["csr", "csr_merge", "coo", "ell", "hybrid", "sellp"])
def test_cgs_convdiff_matches_oracle(g, orc, gen_mod, ctx, fmt):
    A = gen_mod.convdiff2d(40, 0.5)
    n = 1600
    xs = gen_mod.uniform(8, n)
    b = orc.spmv(A, xs)
    rc, xo, info_o = orc.cgs(A, b, tol=1e-10, maxit=2000)
    assert rc == orc.OK
    M = g.Matrix.from_csr(*A).convert(fmt)
    x = dev(np.zeros(n))
    info = g.cgs(M, dev(b), x, tol=1e-10, maxit=2000)
    assert info["status"] == g.OK, info
    # no closed form for CGS iteration counts: they must stay close
    assert abs(info["iterations"] - info_o["iters"]) <= max(3, info_o["iters"] // 10), (info, info_o)
    xg = host(x)
    true = relres(orc, A, b, xg)
    assert true <= 1e-9 and abs(info["true_rel_residual"] - true) <= 1e-12
    assert np.linalg.norm(xg - xo) / np.linalg.norm(xo) <= 1e-6


def test_cgs_identity_and_breakdown(g, gen_mod, ctx):
    b = gen_mod.uniform(3, 10)
    I = g.Matrix.from_csr(np.arange(11, dtype=np.int32), np.arange(10, dtype=np.int32),
                          np.full(10, 2.5))
    x = dev(np.zeros(10))
    info = g.cgs(I, dev(b), x)
    assert info["status"] == g.OK and info["iterations"] == 1
    assert np.allclose(host(x), b / 2.5, rtol=1e-15, atol=0)
    B = g.Matrix.from_csr(np.array([0, 1, 2], np.int32), np.array([1, 0], np.int32), np.ones(2))
    assert g.cgs(B, dev(np.array([1.0, 0.0])), dev(np.zeros(2)))["status"] == g.ERR_BREAKDOWN
    L = g.Matrix.from_csr(*gen_mod.convdiff2d(20, 0.5))
    info = g.cgs(L, dev(np.ones(400)), dev(np.zeros(400)), maxit=3)
    assert info["status"] == g.ERR_NOT_CONVERGED and info["iterations"] == 3
    assert g.cgs(L, dev(np.zeros(400)), dev(np.ones(400)))["status"] == g.OK


# --------------------------------------------------------------------------- GMRES
@pytest.mark.parametrize("fmt", ["csr", "coo", "hybrid", "sellp"])
def test_gmres_convdiff_matches_oracle(g, orc, gen_mod, ctx, fmt):
    A = gen_mod.convdiff2d(40, 0.5)
    n = 1600
    xs = gen_mod.uniform(8, n)
    b = orc.spmv(A, xs)
    rc, xo, info_o = orc.gmres(A, b, tol=1e-10, maxit=20000, m=20)
    assert rc == orc.OK
    ctx.set_solver_opts(krylov_dim=20)
    M = g.Matrix.from_csr(*A).convert(fmt)
    x = dev(np.zeros(n))
    info = g.gmres(M, dev(b), x, tol=1e-10, maxit=20000)
    assert info["status"] == g.OK, info
    # classical Gram-Schmidt (twice when needed) against the oracle's modified
    # Gram-Schmidt: the same Krylov spaces, different rounding
    assert abs(info["iterations"] - info_o["iters"]) <= max(3, info_o["iters"] // 20), (info, info_o)
    assert abs(info["outer_iterations"] - info_o["cycles"]) <= 1
    xg = host(x)
    assert relres(orc, A, b, xg) <= 1e-10
    assert abs(info["true_rel_residual"] - relres(orc, A, b, xg)) <= 1e-13
    assert np.linalg.norm(xg - xo) / np.linalg.norm(xo) <= 1e-7


def test_gmres_minimal_residual_steps(g, orc, ctx):
    """k steps without restart: the residual is the least-squares minimum over
    the Krylov space (numpy on an orthonormal Krylov basis), and x matches
    the oracle's k-step iterate."""
    rng = np.random.default_rng(23)
    n = 30
    D = np.eye(n) * 2 + rng.uniform(-1, 1, (n, n)) * 0.25
    rp = np.arange(0, n * n + 1, n, dtype=np.int32)
    A = (rp, np.tile(np.arange(n, dtype=np.int32), n), D.ravel())
    b = rng.uniform(-1, 1, n)
    ctx.set_solver_opts(krylov_dim=30)
    M = g.Matrix.from_csr(*A)
    for k in range(1, 7):
        x = dev(np.zeros(n))
        info = g.gmres(M, dev(b), x, tol=1e-15, maxit=k)
        assert info["status"] == g.ERR_NOT_CONVERGED and info["iterations"] == k
        xg = host(x)
        K = np.stack([np.linalg.matrix_power(D, j) @ b for j in range(k)], 1)
        Q, _ = np.linalg.qr(K)
        y, *_ = np.linalg.lstsq(D @ Q, b, rcond=None)
        rmin = np.linalg.norm(b - D @ (Q @ y))
        assert abs(np.linalg.norm(b - D @ xg) - rmin) <= 1e-10 * np.linalg.norm(b), k
        rc, xo, _ = orc.gmres(A, b, tol=1e-15, maxit=k, m=30)
        assert np.linalg.norm(xg - xo) <= 1e-10 * np.linalg.norm(xo), k
        assert abs(info["rel_residual"] - rmin / np.linalg.norm(b)) <= 1e-10


@pytest.mark.parametrize("m", [1, 5, 30, 128])
def test_gmres_restart_lengths_laplace(g, orc, gen_mod, ctx, m):
    """n = 65,536 (64 workgroups of the multi-vector passes), restart lengths
    from GMRES(1) to the largest supported."""
    N = 256 if m >= 30 else 32
    A = gen_mod.laplace2d(N)
    n = N * N
    b = orc.spmv(A, gen_mod.uniform(2, n))
    tol = 1e-8
    rc, xo, info_o = orc.gmres(A, b, tol=tol, maxit=4000, m=m)
    ctx.set_solver_opts(krylov_dim=m)
    M = g.Matrix.from_csr(*A)
    x = dev(np.zeros(n))
    info = g.gmres(M, dev(b), x, tol=tol, maxit=4000)
    assert info["status"] == (g.OK if rc == orc.OK else g.ERR_NOT_CONVERGED), (info, info_o)
    assert abs(info["iterations"] - info_o["iters"]) <= max(3, info_o["iters"] // 20), (info, info_o)
    if rc == orc.OK:
        assert relres(orc, A, b, host(x)) <= tol


@pytest.mark.parametrize("m,maxit", [(5, 20000), (30, 20000), (64, 20000), (8, 37)])
def test_gmres_one_workgroup_matches_multikernel(g, orc, gen_mod, ctx, m, maxit):
    """Small CSR systems (n <= 4096, m <= 64) run the whole GMRES in one
    workgroup launch; the multi-kernel path (single_workgroup = 0) takes the
    same steps: equal iteration and cycle counts up to rounding, both
    solutions within the oracle's tolerance (maxit = 37 stops inside a
    cycle)."""
    A = gen_mod.convdiff2d(60, 0.5)
    n = 3600
    b = orc.spmv(A, gen_mod.uniform(9, n))
    rc, xo, info_o = orc.gmres(A, b, tol=1e-10, maxit=maxit, m=m)
    out = {}
    for single in (1, 0):
        ctx.set_solver_opts(krylov_dim=m, single_workgroup=single)
        M = g.Matrix.from_csr(*A)
        x = dev(np.zeros(n))
        out[single] = (g.gmres(M, dev(b), x, tol=1e-10, maxit=maxit), host(x))
    (i1, x1), (i0, x0) = out[1], out[0]
    want = g.OK if rc == orc.OK else g.ERR_NOT_CONVERGED
    assert i1["status"] == i0["status"] == want, (i1, i0, info_o)
    assert abs(i1["iterations"] - i0["iterations"]) <= max(2, i0["iterations"] // 50), (i1, i0)
    assert abs(i1["iterations"] - info_o["iters"]) <= max(3, info_o["iters"] // 20), (i1, info_o)
    assert abs(i1["outer_iterations"] - i0["outer_iterations"]) <= 1
    if want == g.OK:
        assert relres(orc, A, b, x1) <= 1e-10
        assert np.linalg.norm(x1 - x0) / np.linalg.norm(x0) <= 1e-8
    else:
        assert i1["iterations"] == i0["iterations"] == maxit
        assert np.linalg.norm(x1 - x0) / np.linalg.norm(x0) <= 1e-10
        assert abs(i1["rel_residual"] - i0["rel_residual"]) <= 1e-10


@pytest.mark.parametrize("n", [2, 255, 257, 32768, 32769, 65536, 65537, 131073, 524288, 524289])
def test_gmres_multikernel_sizes(g, orc, gen_mod, ctx, n):
    """The multi-kernel passes at the edges of their workgroup sizes (256, 512
    and 1024 rows per workgroup up to 524,288 rows, then the large-grid
    passes), with a restart length past the 32 basis vectors kept in
    registers and a second cycle: 38 steps are the oracle's, to the bound of
    the k-step comparison above (classical against modified Gram-Schmidt)."""
    A = gen_mod.laplace1d(n)
    b = orc.spmv(A, gen_mod.uniform(17, n))
    ctx.set_solver_opts(krylov_dim=34, single_workgroup=0)
    rc, xo, info_o = orc.gmres(A, b, tol=1e-13, maxit=38, m=34)
    x = dev(np.zeros(n))
    info = g.gmres(g.Matrix.from_csr(*A), dev(b), x, tol=1e-13, maxit=38)
    if n > 2:
        assert info["iterations"] == info_o["iters"] == 38
        assert info["outer_iterations"] == info_o["cycles"] == 2
    assert np.linalg.norm(host(x) - xo) <= 1e-10 * np.linalg.norm(xo)


def test_gmres_statuses(g, gen_mod, ctx):
    d = np.array([1.0, 2.0, 3.0] * 17)[:50]
    Dm = g.Matrix.from_csr(np.arange(51, dtype=np.int32), np.arange(50, dtype=np.int32), d)
    bb = gen_mod.uniform(31, 50)
    x = dev(np.zeros(50))
    info = g.gmres(Dm, dev(bb), x, tol=1e-12)
    assert info["status"] == g.OK and info["iterations"] <= 3
    assert np.allclose(host(x), bb / d, rtol=1e-11, atol=0)
    L = g.Matrix.from_csr(*gen_mod.convdiff2d(20, 0.5))
    info = g.gmres(L, dev(np.zeros(400)), dev(np.ones(400)))
    assert info["status"] == g.OK and info["iterations"] == 0
    info = g.gmres(L, dev(np.ones(400)), dev(np.zeros(400)), maxit=7)
    assert info["status"] == g.ERR_NOT_CONVERGED and info["iterations"] == 7
    bn = np.ones(400)
    bn[5] = np.nan
    assert g.gmres(L, dev(bn), dev(np.zeros(400)))["status"] == g.ERR_BREAKDOWN
    for bad in (0, 129):
        with pytest.raises(g.GkoError):
            ctx.set_solver_opts(krylov_dim=bad)


# --------------------------------------------------------------------------- pipelined CG
@pytest.mark.parametrize("fmt", ["csr", "ell", "sellp", "coo"])
def test_pipecg_laplace2d_matches_oracle(g, orc, gen_mod, ctx, fmt):
    N = 64
    A = gen_mod.laplace2d(N)
    xs = gen_mod.uniform(2, N * N)
    b = orc.spmv(A, xs)
    rc, xo, info_o = orc.pipecg(A, b, tol=1e-10)
    M = g.Matrix.from_csr(*A).convert(fmt)
    x = dev(np.zeros(N * N))
    info = g.pipecg(M, dev(b), x, tol=1e-10, maxit=5000)
    assert info["status"] == g.OK, info
    assert abs(info["iterations"] - info_o["iters"]) <= 2, (info, info_o)
    xg = host(x)
    assert relres(orc, A, b, xg) <= 1e-10
    kappa = (4 + 4 * math.cos(math.pi / (N + 1))) / (4 - 4 * math.cos(math.pi / (N + 1)))
    assert np.linalg.norm(xg - xs) / np.linalg.norm(xs) <= kappa * 1e-10


def test_pipecg_iterates_are_cg_iterates(g, orc, ctx):
    """k steps of the GPU's pipelined CG against the oracle's CG (not its
    pipelined CG): equal in exact arithmetic, with and without block-Jacobi."""
    rng = np.random.default_rng(41)
    n = 40
    G = rng.standard_normal((n, n))
    D = G @ G.T / n + np.eye(n)
    D = (D + D.T) / 2
    A = (np.arange(0, n * n + 1, n, dtype=np.int32), np.tile(np.arange(n, dtype=np.int32), n),
         D.ravel())
    b = rng.uniform(-1, 1, n)
    rc, inv = orc.bj_invert(A, 8)
    M = g.Matrix.from_csr(*A)
    for bs in (0, 8):
        if bs:
            ctx.set_solver_opts(precond=g.PRECOND_BLOCK_JACOBI, block_size=8)
        for k in (1, 2, 3, 5, 10):
            x = dev(np.zeros(n))
            info = g.pipecg(M, dev(b), x, tol=1e-300, maxit=k)
            assert info["iterations"] == k
            r1, xc, _ = orc.cg(A, b, tol=1e-300, maxit=k, **({"bj_inv": inv, "bs": 8} if bs else {}))
            assert np.linalg.norm(host(x) - xc) <= 1e-11 * np.linalg.norm(xc), (bs, k)


def test_pipecg_block_jacobi_mixed_and_statuses(g, orc, gen_mod, ctx):
    N = 24
    A = gen_mod.laplace3d(N)
    n = N ** 3
    b = orc.spmv(A, gen_mod.uniform(5, n))
    rc, inv = orc.bj_invert(A, 8)
    rc, xo, info_o = orc.pipecg(A, b, tol=1e-10, bj_inv=inv)
    M = g.Matrix.from_csr(*A)
    ctx.set_solver_opts(precond=g.PRECOND_BLOCK_JACOBI, block_size=8)
    x = dev(np.zeros(n))
    info = g.pipecg(M, dev(b), x, tol=1e-10)
    assert info["status"] == g.OK and abs(info["iterations"] - info_o["iters"]) <= 2, (info, info_o)
    assert relres(orc, A, b, host(x)) <= 1e-10
    ctx.set_solver_opts(precision=g.PREC_MIXED_IR, precond=g.PRECOND_BLOCK_JACOBI, block_size=8)
    x = dev(np.zeros(n))
    info = g.pipecg(M, dev(b), x, tol=1e-10)
    assert info["status"] == g.OK and info["outer_iterations"] >= 2
    assert relres(orc, A, b, host(x)) <= 1e-10
    ctx.set_solver_opts()
    L = g.Matrix.from_csr(*gen_mod.laplace2d(32))
    info = g.pipecg(L, dev(np.zeros(1024)), dev(np.ones(1024)))
    assert info["status"] == g.OK and info["iterations"] == 0
    info = g.pipecg(L, dev(np.ones(1024)), dev(np.zeros(1024)), tol=1e-10, maxit=5)
    assert info["status"] == g.ERR_NOT_CONVERGED and info["iterations"] == 5
    D = g.Matrix.from_csr(np.arange(5, dtype=np.int32), np.arange(4, dtype=np.int32),
                          np.array([1.0, 2.0, -1.0, 3.0]))
    rc, xd, info_d = orc.pipecg((np.arange(5, dtype=np.int32), np.arange(4, dtype=np.int32),
                                 np.array([1.0, 2.0, -1.0, 3.0])), np.ones(4))
    info = g.pipecg(D, dev(np.ones(4)), dev(np.zeros(4)))
    assert info["status"] == g.ERR_NOT_SPD and info["iterations"] == info_d["iters"]


# --------------------------------------------------------------------------- mid-size iterations
def band_spd(n, h):
    """2h + 1 diagonals of -1 around 2h + 1.5: symmetric, row sums >= 1.5."""
    off = np.arange(-h, h + 1)
    c = np.arange(n)[:, None] + off
    ok = (c >= 0) & (c < n)
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(ok.sum(1))
    v = np.where(off == 0, 2 * h + 1.5, -1.0) * np.ones((n, 1))
    return rp, c[ok].astype(np.int32), v[ok]


@pytest.mark.parametrize("n,h,fmt", [
    (1, 0, "csr"), (40, 1, "ell"), (1023, 1, "sellp"), (1025, 1, "csr"), (1024, 1, "csr_merge"),
    (2049, 10, "csr"), (2049, 10, "ell"), (2047, 10, "sellp"), (1025, 30, "csr"), (1500, 60, "csr"),
    (262144, 1, "ell"), (262145, 1, "csr"), (300001, 1, "sellp"), (70000, 10, "csr"), (40000, 30, "csr")])
def test_midsize_iterations_match_oracle(g, orc, gen_mod, ctx, n, h, fmt):
    """The few-kernel iterations of mid-size systems: rows around the 1024 of a
    workgroup and the 256 workgroups of a grid, 1, 4, 8 and 32 lanes per CSR
    row, rows longer than the 8 entries loaded ahead, odd check_every.  The
    k-step iterates are the oracle's.  The matrix has condition at most 4h + 2
    (Gershgorin) and k is small, so rounding differences stay near k kappa u
    for CG (1e-11) and are squared by CGS's polynomial (1e-9)."""
    A = band_spd(n, h)
    b = orc.spmv(A, gen_mod.uniform(19, n))
    M = g.Matrix.from_csr(*A).convert(fmt)
    for solver, k, bound in (("cg", 13, 1e-11), ("fcg", 13, 1e-11), ("pipecg", 9, 1e-11),
                             ("bicgstab", 7, 1e-9), ("cgs", 5, 1e-9)):
        k = min(k, max(1, n // 3))
        ctx.set_solver_opts(check_every=5, single_workgroup=0)
        rc, xo, info_o = getattr(orc, solver)(A, b, tol=1e-14, maxit=k)
        x = dev(np.zeros(n))
        info = getattr(g, solver)(M, dev(b), x, tol=1e-14, maxit=k)
        assert info["iterations"] == info_o["iters"], (solver, info, info_o)
        assert np.linalg.norm(host(x) - xo) <= bound * np.linalg.norm(xo), solver
    for bs in (1, 2, 4, 8, 16):
        rc, inv = orc.bj_invert(A, bs)
        rc, xo, info_o = orc.cg(A, b, tol=1e-14, maxit=min(6, n), bj_inv=inv, bs=bs)
        ctx.set_solver_opts(check_every=5, precond=g.PRECOND_BLOCK_JACOBI, block_size=bs)
        x = dev(np.zeros(n))
        info = g.cg(M, dev(b), x, tol=1e-14, maxit=min(6, n))
        assert np.linalg.norm(host(x) - xo) <= 1e-11 * np.linalg.norm(xo), bs


@pytest.mark.parametrize("h", [1, 5, 13])
@pytest.mark.parametrize("fmt", ["csr", "ell", "sellp"])
def test_large_iterations_match_oracle(g, orc, gen_mod, ctx, h, fmt):
    """Iterations above the mid-size limits, whose products take the columns of
    a banded matrix from its repeated rows (row lengths of 3, 11 and 27: a lane
    and four lanes per CSR row).  Bounds as for the mid-size iterations."""
    n = 2_100_001 if h < 13 else 560_003
    A = band_spd(n, h)
    b = orc.spmv(A, gen_mod.uniform(19, n))
    M = g.Matrix.from_csr(*A).convert(fmt)
    ctx.set_solver_opts(check_every=4, single_workgroup=0)
    for solver, k, bound in (("cg", 6, 1e-11), ("bicgstab", 4, 1e-9), ("cgs", 3, 1e-9), ("pipecg", 5, 1e-11)):
        rc, xo, info_o = getattr(orc, solver)(A, b, tol=1e-14, maxit=k)
        x = dev(np.zeros(n))
        info = getattr(g, solver)(M, dev(b), x, tol=1e-14, maxit=k)
        assert info["iterations"] == info_o["iters"], (solver, info, info_o)
        assert np.linalg.norm(host(x) - xo) <= bound * np.linalg.norm(xo), solver


@pytest.mark.parametrize("maxit", [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 64, 65])
@pytest.mark.parametrize("solver", ["cg", "pipecg", "bicgstab", "cgs"])
def test_caps_at_polling_intervals(g, orc, gen_mod, ctx, solver, maxit):
    """Iteration caps around multiples of the 16 iterations between two looks at
    the state: intervals are enqueued before the state of the one before is
    known, and none may go past the cap or past convergence.  The matrix has
    condition at most 6, so the bounds are those of the mid-size iterations
    times the longer run (5 k u kappa, squared for CGS and BiCGSTAB)."""
    A = band_spd(3001, 1)
    b = orc.spmv(A, gen_mod.uniform(19, 3001))
    M = g.Matrix.from_csr(*A).convert("ell")
    ctx.set_solver_opts(single_workgroup=0)
    rc, xo, info_o = getattr(orc, solver)(A, b, tol=1e-9, maxit=maxit)
    x = dev(np.zeros(3001))
    info = getattr(g, solver)(M, dev(b), x, tol=1e-9, maxit=maxit)
    assert abs(info["iterations"] - info_o["iters"]) <= (0 if info_o["iters"] == maxit else 1)
    assert info["iterations"] <= maxit
    bound = 1e-10 if info["iterations"] == info_o["iters"] else 1e-8
    assert np.linalg.norm(host(x) - xo) <= bound * np.linalg.norm(xo)


# --------------------------------------------------------------------------- shared edge cases
def test_nonzero_initial_guess_and_long_restart(g, orc, gen_mod, ctx):
    A = gen_mod.convdiff2d(30, 0.5)
    n = 900
    b = orc.spmv(A, gen_mod.uniform(8, n))
    x0 = gen_mod.uniform(12, n)
    M = g.Matrix.from_csr(*A)
    ctx.set_solver_opts(krylov_dim=25)
    rc, xo, info_o = orc.gmres(A, b, x0=x0, tol=1e-10, maxit=5000, m=25)
    x = dev(x0.copy())
    info = g.gmres(M, dev(b), x, tol=1e-10, maxit=5000)
    assert info["status"] == g.OK and abs(info["iterations"] - info_o["iters"]) <= max(3, info_o["iters"] // 20)
    assert relres(orc, A, b, host(x)) <= 1e-10
    rc, xo, info_o = orc.cgs(A, b, x0=x0, tol=1e-10, maxit=2000)
    x = dev(x0.copy())
    info = g.cgs(M, dev(b), x, tol=1e-10, maxit=2000)
    assert info["status"] == g.OK and abs(info["iterations"] - info_o["iters"]) <= max(3, info_o["iters"] // 10)
    # restart length above n: the Krylov space becomes invariant (h_{j+1,j} = 0)
    rng = np.random.default_rng(5)
    D = rng.uniform(-1, 1, (40, 40)) + 4 * np.eye(40)
    Ad = (np.arange(0, 1601, 40, dtype=np.int32), np.tile(np.arange(40, dtype=np.int32), 40), D.ravel())
    ctx.set_solver_opts(krylov_dim=128)
    bd = rng.uniform(-1, 1, 40)
    x = dev(np.zeros(40))
    info = g.gmres(g.Matrix.from_csr(*Ad), dev(bd), x, tol=1e-12)
    assert info["status"] == g.OK and info["iterations"] <= 40 and info["outer_iterations"] <= 2
    assert np.linalg.norm(D @ host(x) - bd) <= 1e-11 * np.linalg.norm(bd)


@pytest.mark.parametrize("solver", ["fcg", "pipecg", "cgs", "gmres"])
def test_solver_argument_checks(g, gen_mod, ctx, solver):
    import torch
    fn = getattr(g, solver)
    A = gen_mod.laplace2d(8)
    F = g.Matrix.from_csr(*A, dtype=torch.float32)
    with pytest.raises(g.GkoError) as e:
        fn(F, dev(np.ones(64)), dev(np.zeros(64)), raise_on_failure=True)
    assert e.value.status == g.ERR_UNSUPPORTED          # solvers take FP64 matrices
    R = g.Matrix.from_csr(np.array([0, 1, 2], np.int32), np.array([0, 2], np.int32), np.ones(2),
                          n_cols=3)
    with pytest.raises(g.GkoError) as e:
        fn(R, dev(np.ones(2)), dev(np.zeros(3)), raise_on_failure=True)
    assert e.value.status == g.ERR_DIM_MISMATCH
    M = g.Matrix.from_csr(*A)
    for tol in (0.0, float("inf")):
        with pytest.raises(g.GkoError) as e:
            fn(M, dev(np.ones(64)), dev(np.zeros(64)), tol=tol, raise_on_failure=True)
        assert e.value.status == g.ERR_INVALID_ARG


# ----------------------------------------------------------------- HIP graphs
def _solve_pair(g, ctx, solver, M, b, n, **opts):
    """The same solve with the polling interval replayed from a HIP graph and
    launched kernel by kernel: x and the iteration count."""
    out = []
    for graphs in (1, 0):
        ctx.set_solver_opts(graphs=graphs, single_workgroup=0, **opts)
        x = dev(np.zeros(n))
        info = getattr(g, solver)(M, dev(b), x, tol=1e-10, maxit=5000)
        out.append((host(x), info))
    return out


@pytest.mark.parametrize("fmt", ["csr", "csr_merge", "coo", "ell", "hybrid", "sellp"])
@pytest.mark.parametrize("solver", ["cg", "fcg", "pipecg"])
def test_graph_replay_matches_eager_spd(g, orc, gen_mod, ctx, solver, fmt):
    """CG, flexible and pipelined CG: the graph holds the eager path's kernels
    with the same arguments, so every replay (one per polling interval, with
    the host's convergence poll between them) gives the same bits."""
    A = gen_mod.laplace2d(100)
    n = 10000
    b = orc.spmv(A, gen_mod.uniform(21, n))
    M = g.Matrix.from_csr(*A).convert(fmt)
    (xg, ig), (xe, ie) = _solve_pair(g, ctx, solver, M, b, n, check_every=7)
    assert ig["status"] == g.OK and ie["status"] == g.OK
    assert ig["iterations"] == ie["iterations"] and ig["iterations"] > 7 * 10
    assert np.array_equal(xg, xe)
    assert relres(orc, A, b, xg) <= 1e-10


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
def test_graph_replay_matches_eager_pcg(g, orc, gen_mod, ctx, mixed):
    A = gen_mod.laplace3d(24)
    n = 24 ** 3
    b = orc.spmv(A, gen_mod.uniform(22, n))
    M = g.Matrix.from_csr(*A).convert("sellp")
    (xg, ig), (xe, ie) = _solve_pair(
        g, ctx, "cg", M, b, n, precond=g.PRECOND_BLOCK_JACOBI, block_size=8,
        precision=g.PREC_MIXED_IR if mixed else g.PREC_FP64)
    assert ig["status"] == g.OK and ie["status"] == g.OK
    assert ig["iterations"] == ie["iterations"]
    assert ig["outer_iterations"] == ie["outer_iterations"]
    assert np.array_equal(xg, xe)


@pytest.mark.parametrize("fmt", ["csr", "coo", "ell", "sellp"])
@pytest.mark.parametrize("solver", ["bicgstab", "cgs"])
def test_graph_replay_matches_eager_nonsymmetric(g, orc, gen_mod, ctx, solver, fmt):
    A = gen_mod.convdiff2d(100, 0.5)
    n = 10000
    b = orc.spmv(A, gen_mod.uniform(23, n))
    M = g.Matrix.from_csr(*A).convert(fmt)
    (xg, ig), (xe, ie) = _solve_pair(g, ctx, solver, M, b, n)
    assert ig["status"] == g.OK and ie["status"] == g.OK
    assert ig["iterations"] == ie["iterations"]
    assert np.array_equal(xg, xe)
    assert relres(orc, A, b, xg) <= 1e-9


def test_graphs_option_validated(g, ctx):
    with pytest.raises(g.GkoError) as e:
        ctx.set_solver_opts(graphs=2)
    assert e.value.status == g.ERR_INVALID_ARG
    assert ctx.solver_opts()["graphs"] == 1


# --------------------------------------------------------------------------- what a solve costs behind its end
def scattered(n, per, dominance):
    """Rows of about per + 1 entries, -1 in random columns and a diagonal of
    `dominance` times the others' sum, made on the device."""
    import torch
    r = torch.Generator(device="cuda").manual_seed(n + per)
    i = torch.arange(n, device="cuda")
    j = torch.randint(0, n, (n, per), generator=r, device="cuda")
    key = torch.unique(torch.cat([(i[:, None] * n + j).reshape(-1), i * (n + 1)]))
    row, col = key // n, key % n
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(row, minlength=n), 0, out=rp[1:])
    others = (rp[1:] - rp[:-1] - 1).clamp(min=1).double()
    val = torch.where(row == col, dominance * others[row], torch.full_like(row, -1).double())
    return rp.int(), col.int(), val


def best_of(runs, f):
    import time

    import torch
    best = float("inf")
    for _ in range(runs):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("n,graphs", [(600_001, 1), (600_001, 0), (500_001, 1), (500_001, 0)])
def test_gmres_products_behind_a_cycles_end(g, ctx, n, graphs):
    """A cycle of up to 128 steps that ends after a few, on systems whose
    product (18 million scattered entries) takes much longer than enqueuing a
    step: the solve takes no more products than the polling interval of 16
    steps has, as seen from its time (40 products and 4 ms are allowed; all 128
    would be three times that)."""
    import torch
    M = g.Matrix.from_csr(*scattered(n, 30, 4.0))
    b = torch.rand(n, dtype=torch.float64, device="cuda")
    x, y = torch.zeros_like(b), torch.empty_like(b)
    ctx.set_solver_opts(krylov_dim=128, graphs=graphs)

    def products():
        for _ in range(16):
            g.spmv(M, 1.0, b, 0.0, y)

    def solve():
        x.zero_()
        return g.gmres(M, b, x, tol=1e-3, maxit=500)

    info = solve()
    assert info["status"] == g.OK and info["iterations"] < 16 and info["true_rel_residual"] <= 1e-3
    assert best_of(3, solve) <= best_of(3, products) * 40 / 16 + 0.004


class counting_context:
    """A context whose allocator notes the bytes of every buffer handed out."""

    def __init__(self, g):
        import torch
        self.ctx, self.sizes, device = g.Context(use_torch_allocator=False), [], torch.cuda.current_device()

        def alloc(nbytes, stream, user):
            self.sizes.append(nbytes)
            return torch.cuda.caching_allocator_alloc(int(nbytes), device, stream or 0)

        def dealloc(p, stream, user):
            torch.cuda.caching_allocator_delete(p)

        self.ctx._cbs = (g.ALLOC_FN(alloc), g.DEALLOC_FN(dealloc))
        assert g._lib.gko_context_set_allocator(self.ctx.handle, self.ctx._cbs[0], self.ctx._cbs[1], None) == g.OK


@pytest.mark.parametrize("N,m,one", [(16, 44, True), (20, 50, True), (26, 40, True), (45, 20, True), (64, 10, True),
                                     (64, 12, False), (45, 24, False), (15, 64, False), (32, 50, False)])
def test_gmres_one_workgroup_where_it_is_faster(g, orc, gen_mod, N, m, one):
    """Which cycles run on one workgroup, as seen from the buffers of the solve
    (those that do need no partial sums): those whose steps take it less time
    than the passes over many workgroups, few rows with up to 50 steps a cycle
    but 4,096 rows only up to about 10.  Two full cycles match the oracle on
    either path."""
    A = gen_mod.convdiff2d(N, 0.5)
    n = N * N
    b = gen_mod.uniform(5, n)
    rc, xo, _ = orc.gmres(A, b, tol=1e-30, maxit=2 * m, m=m)
    c = counting_context(g)
    M, held = g.Matrix.from_csr(*A, ctx=c.ctx), {}
    for single in (1, 0):
        c.ctx.set_solver_opts(krylov_dim=m, single_workgroup=single)
        x = dev(np.zeros(n))
        c.sizes.clear()
        info = g.gmres(M, dev(b), x, tol=1e-30, maxit=2 * m)
        held[single] = sorted(c.sizes)
        assert info["status"] == g.ERR_NOT_CONVERGED and info["iterations"] == 2 * m, info
        assert np.linalg.norm(host(x) - xo) <= 1e-9 * np.linalg.norm(xo)
    assert (sum(held[1]) < sum(held[0])) if one else held[1] == held[0], held


@pytest.mark.parametrize("solver,fmt,block", [("cg", "coo", 0), ("bicgstab", "hybrid", 0), ("cgs", "csr", 0),
                                              ("fcg", "csr_merge", 0), ("pipecg", "csr", 4)])
def test_products_behind_a_solves_end(g, ctx, solver, fmt, block):
    """A solve that ends in its second polling interval, on a system whose
    product (18 million scattered entries) does not return at once behind the
    end: with graphs it takes as many products as without, two intervals, as
    seen from the times (a quarter is allowed; a third interval would be a
    half)."""
    import torch
    n = 300_001
    rp, col, val = scattered(n, 30, 1.5)
    key = torch.repeat_interleave(torch.arange(n, device="cuda"), (rp[1:] - rp[:-1]).long()) * n + col
    if solver != "bicgstab" and solver != "cgs":              # symmetric: A + A^T
        both = torch.cat([key, key % n * n + key // n])
        key, place = torch.unique(both, return_inverse=True)
        val = torch.zeros(key.numel(), dtype=torch.float64, device="cuda").index_add_(0, place, torch.cat([val, val]))
        rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(torch.bincount(key // n, minlength=n), 0, out=rp[1:])
        row, col = key // n, (key % n)
        others = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, row, torch.where(row == col, 0.0, -val))
        val = torch.where(row == col, 1.5 * others[row], val)
        rp, col = rp.int(), col.int()
    M = g.Matrix.from_csr(rp, col, val).convert(fmt)
    b = torch.rand(n, dtype=torch.float64, device="cuda")
    x = torch.zeros_like(b)
    pre = dict(precond=g.PRECOND_BLOCK_JACOBI, block_size=block) if block else {}

    def solve():
        x.zero_()
        return getattr(g, solver)(M, b, x, tol=1e-9, maxit=500)

    ctx.set_solver_opts(graphs=0, **pre)
    k = solve()["iterations"]
    times = []
    for graphs in (0, 1):
        ctx.set_solver_opts(graphs=graphs, check_every=k // 2 + 1, **pre)
        info = solve()
        assert info["status"] == g.OK and info["iterations"] == k
        times.append(best_of(5, solve))
    assert times[1] <= 1.25 * times[0], (k, times)


# --------------------------------------------------------------------------- which systems take the mid-size kernels
@pytest.mark.parametrize("solver,products", [("cg", 1), ("bicgstab", 2), ("cgs", 2)])
def test_iterations_on_scattered_columns(g, ctx, solver, products):
    """A million rows of 9 scattered entries, whose gathers miss the caches: an
    iteration takes less than twice its products (it took 2.9 to 3.6 times them
    where two or three vectors were gathered for each entry)."""
    import torch
    n = 1_000_000
    M = g.Matrix.from_csr(*scattered(n, 8, 1.02))
    b = torch.rand(n, dtype=torch.float64, device="cuda")
    x, y = torch.zeros_like(b), torch.empty_like(b)

    def product():
        for _ in range(20):
            g.spmv(M, 1.0, b, 0.0, y)

    def solve():
        x.zero_()
        return getattr(g, solver)(M, b, x, tol=1e-30, maxit=16)

    info = solve()
    assert info["iterations"] == 16
    assert best_of(3, solve) / 16 <= 2 * products * best_of(3, product) / 20


@pytest.mark.parametrize("n", [50_000, 200_000])
def test_iterations_with_a_few_long_rows(g, ctx, n):
    """CSR rows of 5 entries, ten of them with 240: one lane may not walk a long
    row while its workgroup waits.  The iteration takes at most 0.8 of SELL-P's,
    whose long rows are walked by a thread (0.97 and 0.90 where CSR's were)."""
    import torch
    rng = torch.Generator(device="cuda").manual_seed(3)
    i = torch.arange(n, device="cuda")
    key = [i * (n + 1)]
    for d in (1, 2):
        key += [i[:-d] * n + i[:-d] + d, i[d:] * n + i[d:] - d]
    hub = torch.randperm(n, generator=rng, device="cuda")[:10].repeat_interleave(240)
    far = torch.randint(0, n, (2400,), generator=rng, device="cuda")
    key = torch.unique(torch.cat(key + [hub * n + far, far * n + hub]))
    row, col = key // n, key % n
    lens = torch.bincount(row, minlength=n)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=rp[1:])
    val = torch.where(row == col, 1.02 * (lens[row] - 1).double(), torch.full_like(row, -1).double())
    M = g.Matrix.from_csr(rp.int(), col.int(), val)
    b = torch.rand(n, dtype=torch.float64, device="cuda")
    x = torch.zeros_like(b)
    times = []
    for fmt in ("csr", "sellp"):
        M.convert(fmt)

        def solve():
            x.zero_()
            return g.cg(M, b, x, tol=1e-30, maxit=32)

        assert solve()["iterations"] == 32
        times.append(best_of(5, solve))
    assert times[0] <= 0.8 * times[1], times


@pytest.mark.parametrize("n,per,fmt", [(1500, 6, "csr"), (40_000, 6, "csr"), (40_000, 6, "ell"), (40_000, 3, "sellp"),
                                       (65_536, 8, "csr"), (65_537, 8, "csr"), (90_000, 14, "csr"), (30_000, 30, "csr"),
                                       (20_000, 14, "ell"), (250_000, 6, "csr_merge")])
def test_scattered_systems_match_oracle(g, orc, gen_mod, ctx, n, per, fmt):
    """Symmetric matrices with scattered columns on either side of the rule that
    sends a solve to the mid-size kernels, with one and with four lanes per CSR
    row: the k-step iterates are the oracle's.  Diagonally dominant by a half, so
    the condition is at most 5 (Gershgorin); bounds as for the banded systems."""
    rng = np.random.default_rng(n + per)
    i, j = (rng.integers(0, n, n * per // 2) for _ in range(2))
    key = np.unique(np.concatenate([i * n + j, j * n + i, np.arange(n) * (n + 1)]))
    row, col = key // n, key % n
    lens = np.bincount(row, minlength=n)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    val = np.where(row == col, 1.5 * np.maximum(lens[row] - 1, 1), -1.0)
    A = (rp, col.astype(np.int32), val)
    b = orc.spmv(A, gen_mod.uniform(23, n))
    M = g.Matrix.from_csr(*A).convert(fmt)
    ctx.set_solver_opts(check_every=5, single_workgroup=0)
    for solver, k, bound in (("cg", 11, 1e-11), ("fcg", 11, 1e-11), ("pipecg", 9, 1e-11), ("bicgstab", 5, 1e-9),
                             ("cgs", 4, 1e-9)):
        rc, xo, info_o = getattr(orc, solver)(A, b, tol=1e-14, maxit=k)
        x = dev(np.zeros(n))
        info = getattr(g, solver)(M, dev(b), x, tol=1e-14, maxit=k)
        assert info["iterations"] == info_o["iters"] == k, (solver, info, info_o)
        assert np.linalg.norm(host(x) - xo) <= bound * np.linalg.norm(xo), solver


@pytest.mark.parametrize("solver", ["cg", "fcg"])
@pytest.mark.parametrize("fmt,second", [("csr", True), ("sellp", True), ("coo", False)])
def test_second_direction_held_where_it_is_used(g, gen_mod, solver, fmt, second):
    """A CG solve holds a second direction vector only where the kernels that
    alternate between two run: on a COO matrix it holds r, p and q."""
    N = 150
    n = N * N
    c = counting_context(g)
    M = g.Matrix.from_csr(*gen_mod.laplace2d(N), ctx=c.ctx)
    M.convert(fmt)
    b, x = dev(gen_mod.uniform(6, n)), dev(np.zeros(n))
    c.sizes.clear()
    info = getattr(g, solver)(M, b, x, tol=1e-8, maxit=2000)
    assert info["status"] == g.OK and info["true_rel_residual"] <= 1e-8, info
    assert sum(z == 8 * n for z in c.sizes) == (4 if second else 3), sorted(c.sizes)
