"""GPU parity of the SpMV family and the format conversions against the oracle.

SpMV (Sec. 6.1): every format, FP64 and FP32, on edge cases (empty rows and
runs of them, nnz = 0, a single dense row, rows much longer than a tile or a
chunk, rectangular shapes) and on small instances of the workload shapes.
Conversions are integer bookkeeping and must match the oracle's arrays byte
for byte."""
import numpy as np
import pytest

from gpu_util import assert_spmv_close, dev, host, tiny_cases, workload_cases

pytestmark = pytest.mark.gpu

FORMATS = ["csr", "csr_merge", "coo", "ell", "hybrid", "sellp"]


@pytest.fixture(scope="module")
def g():
    import paper_2011_08879_amd as g
    return g


@pytest.fixture(scope="module")
def cases(gen_mod):
    c = tiny_cases()
    c.update(workload_cases(gen_mod))
    return c


def make(g, case, f32=False):
    n, m, rp, col, val = case
    import torch
    return g.Matrix.from_csr(rp, col, val.astype(np.float32) if f32 else val, n_cols=m,
                             dtype=torch.float32 if f32 else torch.float64)


def ell_infeasible(case, vb=8):
    """The library refuses ELL when padded storage exceeds 4x the CSR storage."""
    n, m, rp, col, val = case
    K = int(np.diff(rp).max(initial=0))
    ld = (n + 63) // 64 * 64
    return K * ld * (vb + 4) > 4 * (len(col) * (vb + 4) + (n + 1) * 4)


def sellp_infeasible(case, vb=8):
    """SELL-P is refused by the same rule: padded slots above 4x the CSR storage."""
    n, m, rp, col, val = case
    lens = np.diff(rp).astype(np.int64)
    ns = (n + 63) // 64
    padded = np.zeros(ns * 64, np.int64)
    padded[:n] = lens
    slots = int(padded.reshape(ns, 64).max(axis=1).sum()) * 64 if ns else 0
    return slots * (vb + 4) > 4 * (len(col) * (vb + 4) + (n + 1) * 4)


def infeasible(fmt, case, vb=8):
    return ((fmt == "ell" and ell_infeasible(case, vb)) or
            (fmt == "sellp" and sellp_infeasible(case, vb)))


@pytest.mark.parametrize("f32", [False, True], ids=["f64", "f32"])
@pytest.mark.parametrize("fmt", FORMATS)
def test_spmv_parity(g, orc, gen_mod, cases, fmt, f32):
    import torch
    for name, case in cases.items():
        n, m, rp, col, val = case
        A = make(g, case, f32)
        if infeasible(fmt, case, 4 if f32 else 8):
            with pytest.raises(g.GkoError) as e:
                A.convert(fmt)
            assert e.value.status == g.ERR_UNSUPPORTED
            assert A.describe().format == "csr"
            continue
        A.convert(fmt)
        assert A.describe().format == fmt
        x = gen_mod.uniform(7, m)
        y0 = gen_mod.uniform(8, n)
        if f32:
            vals, x, y0 = (val.astype(np.float32).astype(np.float64), x.astype(np.float32).astype(np.float64),
                           y0.astype(np.float32).astype(np.float64))
        else:
            vals = val
        Ah = (rp, col, vals)
        tdt = torch.float32 if f32 else torch.float64
        lens = np.diff(rp)
        for alpha, beta in [(1.0, 0.0), (1.5, -0.5), (-1.0, 1.0)]:
            xd = dev(x, tdt)
            yd = dev(y0, tdt)
            if beta == 0.0:
                yd.fill_(float("nan"))   # beta = 0: y must not be read
            g.spmv(A, alpha, xd, beta, yd)
            y = host(yd)
            ref = orc.spmv_dot2(Ah, x, alpha, beta, y0)
            absy = orc.spmv_absbound(Ah, x, alpha, beta, y0)
            assert_spmv_close(y, ref, absy, lens, f32, "%s/%s a=%g b=%g" % (name, fmt, alpha, beta))
        A.close()


@pytest.mark.parametrize("fmt", FORMATS)
def test_spmv_deterministic(g, gen_mod, cases, fmt):
    import torch
    case = cases["lognormal_20k"]
    if fmt in ("ell", "sellp"):
        case = cases["stencil27_14"]
    n, m = case[0], case[1]
    A = make(g, case).convert(fmt)
    x = dev(gen_mod.uniform(3, m))
    outs = []
    for _ in range(4):
        y = torch.empty(n, dtype=torch.float64, device="cuda")
        g.spmv(A, 1.0, x, 0.0, y)
        outs.append(host(y).view(np.int64))
    for o in outs[1:]:
        assert np.array_equal(o, outs[0])


def test_spmv_rejects_overlap(g, cases):
    import torch
    A = make(g, cases["laplace2d_64"])
    v = torch.zeros(4096 + 10, dtype=torch.float64, device="cuda")
    with pytest.raises(g.GkoError) as e:
        g.spmv(A, 1.0, v[:4096], 0.0, v[10:])
    assert e.value.status == g.ERR_INVALID_ARG


def test_create_rejects_malformed(g):
    import torch
    rp = np.array([0, 2, 1, 3], np.int32)          # decreasing offsets
    with pytest.raises(g.GkoError):
        g.Matrix.from_csr(rp, np.array([0, 1, 2], np.int32), np.ones(3))
    rp = np.array([0, 2, 3], np.int32)
    with pytest.raises(g.GkoError):                  # unsorted columns in row 0
        g.Matrix.from_csr(rp, np.array([1, 0, 1], np.int32), np.ones(3))
    with pytest.raises(g.GkoError):                  # column out of range
        g.Matrix.from_csr(rp, np.array([0, 1, 7], np.int32), np.ones(3), n_cols=3)
    # int64 row offsets are accepted
    A = g.Matrix.from_csr(np.array([0, 1, 2], np.int64), np.array([0, 1], np.int32), np.ones(2))
    assert A.describe().nnz == 2


def bits(a):
    return np.ascontiguousarray(a).view(np.int64 if a.dtype == np.float64 else np.int32)


@pytest.mark.parametrize("f32", [False, True], ids=["f64", "f32"])
def test_conversions_bit_exact(g, orc, cases, f32):
    for name, case in cases.items():
        n, m, rp, col, val = case
        vals = val.astype(np.float32) if f32 else val
        A = make(g, case, f32)
        Ah = (rp, col, vals.astype(np.float64))
        # COO
        A.convert("coo")
        s = A.export_storage()
        r, c, v = orc.csr_to_coo(Ah)
        assert np.array_equal(host(s["coo_row"]), r), name
        assert np.array_equal(host(s["coo_col"]), c), name
        assert np.array_equal(bits(host(s["coo_val"])), bits(v.astype(vals.dtype))), name
        # HYB
        A.convert("hybrid")
        s = A.export_storage()
        K, ld, ec, ev, tr, tc, tv = orc.csr_to_hyb(Ah, value_bytes=4 if f32 else 8)
        assert (s["K"], s["ld"]) == (K, ld), name
        assert np.array_equal(host(s["ell_col"]), ec), name
        assert np.array_equal(bits(host(s["ell_val"])), bits(ev.astype(vals.dtype))), name
        assert np.array_equal(host(s["coo_row"]), tr), name
        assert np.array_equal(host(s["coo_col"]), tc), name
        assert np.array_equal(bits(host(s["coo_val"])), bits(tv.astype(vals.dtype))), name
        # ELL
        if not ell_infeasible(case, 4 if f32 else 8):
            A.convert("ell")
            s = A.export_storage()
            K, ld, ec, ev = orc.csr_to_ell(Ah)
            assert (s["K"], s["ld"]) == (K, ld), name
            assert np.array_equal(host(s["ell_col"]), ec), name
            assert np.array_equal(bits(host(s["ell_val"])), bits(ev.astype(vals.dtype))), name
        # SELL-P
        if not sellp_infeasible(case, 4 if f32 else 8):
            A.convert("sellp")
            d = A.describe()
            s = A.export_sellp()
            w, sets, sc, sv = orc.csr_to_sellp(Ah)
            assert (s["slice"], d.sellp_slices, d.sellp_slots) == (64, len(w), sets[-1]), name
            assert np.array_equal(host(s["sets"]), sets), name
            assert np.array_equal(host(s["widths"]), w), name
            assert np.array_equal(host(s["col"]), sc), name
            assert np.array_equal(bits(host(s["val"])), bits(sv.astype(vals.dtype))), name
            vb = 4 if f32 else 8
            wide = [int(x) for x in w if x > 512]       # slices summed by column chunks
            items = sum((x + 255) // 256 for x in wide)
            assert d.sellp_wide_slices == len(wide), name
            extra = (len(wide) * 4 + (len(wide) + 1) * 4 + items * (8 + 64 * 8)) if wide else 0
            assert d.stored_bytes == sets[-1] * (vb + 4) + (len(w) + 1) * 8 + len(w) * 4 + extra, name
            B = A.clone()
            assert B.describe() == d
            sb = B.export_sellp()
            assert np.array_equal(host(sb["col"]), sc), name
            B.close()
        # merge, and back to CSR from whatever is stored
        for fmt in ["csr_merge", "coo", "hybrid", "sellp", "csr"]:
            if fmt == "sellp" and sellp_infeasible(case, 4 if f32 else 8):
                continue
            A.convert(fmt)
            erp, ecol, evl = (host(t) for t in A.export_csr())
            assert np.array_equal(erp, rp) and np.array_equal(ecol, col), (name, fmt)
            assert np.array_equal(bits(evl), bits(vals)), (name, fmt)
        d = A.describe()
        assert d.format == "csr" and d.nnz == len(col) and d.stored_bytes == (n + 1) * 4 + len(col) * (8 if f32 else 12)
        B = A.clone()
        assert B.describe() == d
        A.close()
        B.close()


def _edge_lens(name):
    rng = np.random.default_rng(7)
    if name.startswith("even"):             # n rows of l entries: tiles of 64 rows, chunks of 2048 entries
        n, l = (int(v) for v in name[4:].split("x"))
        return np.full(n, l)
    lens = rng.integers(0, 12, 700)
    lens[int(rng.integers(0, 700))] = int(name[4:])   # one row of that length
    return lens


@pytest.mark.parametrize("name", ["even1x1", "even63x3", "even64x32", "even65x32", "even64x33", "even255x5",
                                  "even257x16", "long2047", "long2048", "long2049", "long5000", "long8191",
                                  "long8192", "long9000"])
@pytest.mark.parametrize("f32", [False, True])
def test_conversions_at_tile_and_chunk_edges(g, orc, name, f32):
    """Row tiles (64 and 256 rows) and LDS chunks (2048 entries; 8192 histogram
    bins) at their edges: stored arrays against the oracle's, and back."""
    lens = _edge_lens(name)
    n, m = len(lens), 10000
    rng = np.random.default_rng(11)
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(m, size=l, replace=False)) for l in lens]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(col)).astype(np.float32 if f32 else np.float64)
    case = (n, m, rp, col, vals)
    A = make(g, (n, m, rp, col, vals.astype(np.float64)), f32)
    Ah = (rp, col, vals.astype(np.float64))

    def back(fmt):
        erp, ecol, evl = (host(t) for t in A.convert("csr").export_csr())
        assert np.array_equal(erp, rp) and np.array_equal(ecol, col), fmt
        assert np.array_equal(bits(evl), bits(vals)), fmt

    s = A.convert("coo").export_storage()
    assert np.array_equal(host(s["coo_row"]), np.repeat(np.arange(n), lens))
    back("coo")
    s = A.convert("hybrid").export_storage()
    K, ld, ec, ev, tr, tc, tv = orc.csr_to_hyb(Ah, value_bytes=4 if f32 else 8)
    assert (s["K"], s["ld"]) == (K, ld)
    for key, want in (("ell_col", ec), ("coo_row", tr), ("coo_col", tc)):
        assert np.array_equal(host(s[key]), want), key
    assert np.array_equal(bits(host(s["ell_val"])), bits(ev.astype(vals.dtype)))
    assert np.array_equal(bits(host(s["coo_val"])), bits(tv.astype(vals.dtype)))
    back("hybrid")
    if not ell_infeasible(case, 4 if f32 else 8):
        s = A.convert("ell").export_storage()
        K, ld, ec, ev = orc.csr_to_ell(Ah)
        assert np.array_equal(host(s["ell_col"]), ec)
        assert np.array_equal(bits(host(s["ell_val"])), bits(ev.astype(vals.dtype)))
        back("ell")
    if not sellp_infeasible(case, 4 if f32 else 8):
        s = A.convert("sellp").export_sellp()
        w, sets, sc, sv = orc.csr_to_sellp(Ah)
        assert np.array_equal(host(s["widths"]), w) and np.array_equal(host(s["sets"]), sets)
        assert np.array_equal(host(s["col"]), sc)
        assert np.array_equal(bits(host(s["val"])), bits(sv.astype(vals.dtype)))
        back("sellp")


def _pattern_rows(name):
    """(n, m, rp, col) with at least a million entries whose rows repeat a few lists of column offsets."""
    lists, length, n = (int(v) for v in name.replace("odd", "").split("x"))
    rng = np.random.default_rng(lists * 1000 + length)
    spread = 2 * length + 40
    offs = [np.sort(rng.choice(np.arange(-spread, spread), size=l, replace=False))
            for l in rng.integers(max(0, length - 2), length + 1, lists)]
    offs[0] = np.sort(rng.choice(np.arange(-spread, spread), size=length, replace=False))
    if lists > 2:
        offs[1] = np.zeros(0, np.int64)                      # empty rows
    pat = np.where(np.arange(n) < lists, np.arange(n) % lists, rng.integers(0, lists, n))
    m = n + 2 * spread                                       # every list fits in every row
    lens = np.array([len(o) for o in offs])[pat]
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(lens)
    padded = np.zeros((lists, length), np.int64)
    for k, o in enumerate(offs):
        padded[k, :len(o)] = o
    inside = np.arange(length)[None, :] < lens[:, None]
    col = ((np.arange(n) + spread)[:, None] + padded[pat])[inside]
    if name.endswith("odd"):                                 # one more list: a row of its own
        r = n - 70
        col[rp[r]:rp[r + 1]] = np.arange(lens[r])
    assert rp[-1] >= 1_000_000
    return n, m, rp.astype(np.int32), col.astype(np.int32)


@pytest.mark.parametrize("name", ["1x5x230001", "2x8x150079", "27x7x200063", "3x9x180064", "84x12x120065",
                                  "30x13x120001", "35x28x70001", "27x27x60001odd", "127x5x300000", "127x6x300000odd",
                                  "128x4x400001", "128x5x300001odd", "129x5x300001", "1x64x20001", "2x70x20100",
                                  "2x200x10127", "1x256x6001", "3x256x9001"])
def test_repeated_rows(g, orc, name):
    """Matrices whose rows repeat a few lists of column offsets, whose kernels take the columns from a table of
    the lists: the numbers of lists (128) and of table entries (1024) at which that ends, row lengths at the
    sizes that kernels are compiled for (8, 12, 28), rows in the last tile, an empty list, one odd row."""
    n, m, rp, col = _pattern_rows(name)
    rng = np.random.default_rng(5)
    val, lens = rng.uniform(-1, 1, len(col)), np.diff(rp)
    x, y0 = rng.uniform(-1, 1, m), rng.uniform(-1, 1, n)
    for f32 in (False, True):
        t = np.float32 if f32 else np.float64
        A = make(g, (n, m, rp, col, val.astype(t)), f32)
        xs, ys, vs = (v.astype(t).astype(np.float64) for v in (x, y0, val))
        terms = np.append(vs * xs[col], 0.0).astype(np.longdouble)
        want, size = (np.where(lens > 0, np.add.reduceat(v, rp[:-1]), 0.0) for v in (terms, np.abs(terms)))
        want, size = (1.5 * want + 0.5 * ys).astype(np.float64), (1.5 * size + 0.5 * np.abs(ys)).astype(np.float64)
        for fmt in ("csr", "ell", "sellp", "hybrid"):
            C = A.clone().convert(fmt)
            y = dev(y0.astype(t))
            g.spmv(C, 1.5, dev(x.astype(t)), 0.5, y)
            assert_spmv_close(host(y), want, size, lens, f32, "%s %s" % (name, fmt))
            C.close()
        A.close()


def _coo_lens(name):
    rng = np.random.default_rng(len(name))
    kind, n, l = name.split("x")
    n, l = int(n), int(l)
    if kind == "even":
        return np.full(n, l)
    lens = rng.integers(0, l + 1, n)
    if kind == "gaps":                                       # runs of empty rows, also first and last
        lens[:n // 5] = 0
        lens[n // 3:n // 2] = 0
        lens[-(n // 6):] = 0
    return lens


@pytest.mark.parametrize("name", ["evenx1x1", "evenx4x64", "evenx5x64", "evenx4x63", "evenx64x16", "evenx65x16", "evenx33x31",
                                  "evenx256x1", "evenx257x1", "evenx1025x3", "evenx40x65", "evenx7x300", "randx900x64",
                                  "randx900x5", "gapsx2000x12", "gapsx3000x64", "randx3000x66", "randx500x256",
                                  "randx500x300", "evenx46876x64", "gapsx300000x33"])
@pytest.mark.parametrize("f32", [False, True])
def test_coo_rows_at_batch_and_chunk_edges(g, name, f32):
    """COO rows at the ends of batches (64 entries), of a wavefront's chunks (256 and, from 3 million entries on,
    512) and at 64 entries, up to which a wavefront keeps its rows whole; 256, from which on loads go eight deep."""
    lens = _coo_lens(name)
    n, m = len(lens), 1000
    rng = np.random.default_rng(3)
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    start = rng.integers(0, m - 301, n)
    row = np.repeat(np.arange(n), lens)
    col = (start[row] + np.arange(len(row)) - rp[:-1][row]).astype(np.int32)
    t = np.float32 if f32 else np.float64
    val, x, y0 = (rng.uniform(-1, 1, k).astype(t) for k in (len(col), m, n))
    A = make(g, (n, m, rp, col, val), f32).convert("coo")
    terms = np.append(val.astype(np.float64) * x.astype(np.float64)[col], 0.0).astype(np.longdouble)
    at = np.minimum(rp[:-1], len(col))
    sums, size = (np.where(lens > 0, np.add.reduceat(v, at), 0.0) for v in (terms, np.abs(terms)))
    for alpha, beta in ((1.0, 0.0), (-1.5, 0.5)):
        y = dev(y0)
        g.spmv(A, alpha, dev(x), beta, y)
        assert_spmv_close(host(y), (alpha * sums + beta * y0).astype(np.float64),
                          (abs(alpha) * size + beta * np.abs(y0)).astype(np.float64), lens, f32, name)


def test_auto_picks_a_format(g, cases):
    A = make(g, cases["stencil27_14"])
    A.convert("auto")
    assert A.describe().format in g.SELECTOR_FORMATS


def test_sellp_pads_per_slice(g, orc):
    """One long row makes ELL pad every row to it; SELL-P pads only its slice."""
    rng = np.random.default_rng(77)
    n = 3000
    lens = rng.integers(1, 9, n)
    lens[1234] = 100
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(n, size=l, replace=False)) for l in lens]).astype(np.int32)
    val = rng.uniform(-1, 1, len(col))
    case = (n, n, rp, col, val)
    assert ell_infeasible(case) and not sellp_infeasible(case)
    A = make(g, case)
    with pytest.raises(g.GkoError):
        A.convert("ell")
    A.convert("sellp")
    d = A.describe()
    w, sets, sc, sv = orc.csr_to_sellp((rp, col, val))
    assert d.sellp_slots == sets[-1] and d.sellp_slots < 3 * len(col)   # ELL: 22x
    # SELL-P to every other format and back is bit-exact
    for fmt in ["coo", "sellp", "hybrid", "sellp", "csr_merge", "sellp"]:
        A.convert(fmt)
    s = A.export_sellp()
    assert np.array_equal(host(s["col"]), sc) and np.array_equal(bits(host(s["val"])), bits(sv))
    with pytest.raises(g.GkoError) as e:     # not stored as SELL-P
        A.convert("csr")
        A.export_sellp()
    assert e.value.status == g.ERR_INVALID_ARG


def test_csr_kernel_choice_and_parity(g, orc, gen_mod):
    """The CSR kernel follows the row-length rule (the LDS-staged row-per-thread
    kernel, with 1, 4 or 8 lanes per row, for rows of a mean up to 96 and at
    most 256 entries; a quarter-mean subwarp for longer regular rows; a
    mean-width subwarp plus the workgroup-per-row kernel for irregular rows),
    and each of these paths meets the SpMV bound against the oracle."""
    rng = np.random.default_rng(21)
    lens = list(rng.integers(1, 4, 700))
    lens[350] = 300
    rp = np.zeros(701, np.int32)
    rp[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(700, size=l, replace=False)) for l in lens]).astype(np.int32)
    cases = {
        "laplace2d": (gen_mod.laplace2d(40), 0, False),
        "banded_mean64": (gen_mod.banded(12, 3000, 64, 48, 80), 0, False),
        "banded_mean120": (gen_mod.banded(13, 3000, 128, 100, 140), 16, False),
        "banded_mean40": (gen_mod.banded(19, 3000, 40, 32, 48), 0, False),
        "stencil27_19": (gen_mod.stencil27(19), 0, False),
        "lognormal": (gen_mod.random_lognormal(4, 20000, max_len=3000), 16, True),
        "one_long_row": ((rp, col, rng.uniform(-1, 1, len(col))), 4, True),
    }
    for name, (A, kernel, has_long) in cases.items():
        M = g.Matrix.from_csr(*A)
        d = M.describe()
        lens = np.diff(A[0])
        assert d.csr_kernel == kernel, (name, d)
        if kernel == 0:   # lanes per row from the mean row length
            mean = len(A[1]) / (len(A[0]) - 1)
            assert d.csr_row_lanes == (8 if mean >= 56 else 4 if mean >= 12 else 1), (name, d)
        assert d.max_row_len == lens.max(), (name, d)
        assert (d.csr_long_rows > 0) == has_long, (name, d)
        if has_long:
            assert d.csr_long_rows == int((lens > max(4 * kernel, 64)).sum()), (name, d)
        n = len(A[0]) - 1
        x = gen_mod.uniform(7, n)
        y = dev(np.full(n, np.nan))
        g.spmv(M, 1.0, dev(x), 0.0, y)
        ref = orc.spmv_dot2(A, x, 1.0, 0.0, np.zeros(n))
        absy = orc.spmv_absbound(A, x, 1.0, 0.0, np.zeros(n))
        assert_spmv_close(host(y), ref, absy, lens, False, name)
        M.close()


def arrow_matrix(n, arms, seed):
    """SPD: diagonal 4 + |row degree|, a tridiagonal band, and rows/columns
    0..len(arms)-1 coupled to `arms[k]` random far columns (a few long rows)."""
    rng = np.random.default_rng(seed)
    ent = {}
    for i in range(n):
        for j in (i - 1, i + 1):
            if 0 <= j < n:
                ent[(i, j)] = -1.0
    for k, a in enumerate(arms):
        for j in rng.choice(np.arange(len(arms), n), size=a, replace=False):
            v = rng.uniform(-0.5, 0.5)
            ent[(k, int(j))] = v
            ent[(int(j), k)] = v
    rows = [[] for _ in range(n)]
    for (i, j), v in ent.items():
        rows[i].append((j, v))
    rp, col, val = [0], [], []
    for i in range(n):
        r = sorted(rows[i])
        diag = 4.0 + sum(abs(v) for _, v in r)
        r = sorted(r + [(i, diag)])
        col += [j for j, _ in r]
        val += [v for _, v in r]
        rp.append(len(col))
    return np.array(rp, np.int32), np.array(col, np.int32), np.array(val)


@pytest.mark.parametrize("f32", [False, True], ids=["f64", "f32"])
def test_sellp_wide_slices(g, orc, gen_mod, f32):
    """Slices made wide by a few long rows are summed by column chunks: parity
    of the product, an unchanged layout, and CG through the unfused path."""
    import torch
    n = 20000
    rp, col, val = arrow_matrix(n, [3000, 700, 1500], 5)
    case = (n, n, rp, col, val)
    assert not sellp_infeasible(case, 4 if f32 else 8)
    A = make(g, case, f32).convert("sellp")
    d = A.describe()
    assert d.sellp_wide_slices == 1                  # rows 0-2 share the first slice
    vals = val.astype(np.float32).astype(np.float64) if f32 else val
    w, sets, sc, sv = orc.csr_to_sellp((rp, col, vals))
    s = A.export_sellp()
    assert np.array_equal(host(s["col"]), sc) and np.array_equal(host(s["sets"]), sets)
    x = gen_mod.uniform(7, n)
    y0 = gen_mod.uniform(8, n)
    if f32:
        x, y0 = x.astype(np.float32).astype(np.float64), y0.astype(np.float32).astype(np.float64)
    tdt = torch.float32 if f32 else torch.float64
    for alpha, beta in [(1.0, 0.0), (1.5, -0.5)]:
        yd = dev(y0, tdt)
        g.spmv(A, alpha, dev(x, tdt), beta, yd)
        ref = orc.spmv_dot2((rp, col, vals), x, alpha, beta, y0)
        absy = orc.spmv_absbound((rp, col, vals), x, alpha, beta, y0)
        assert_spmv_close(host(yd), ref, absy, np.diff(rp), f32, "arrow/sellp")
    if not f32:
        b = orc.spmv((rp, col, val), gen_mod.uniform(2, n))
        rc, xo, info_o = orc.cg((rp, col, val), b, tol=1e-10)
        xg = dev(np.zeros(n))
        info = g.cg(A, dev(b), xg, tol=1e-10)
        assert info["status"] == g.OK and abs(info["iterations"] - info_o["iters"]) <= 2
        assert np.linalg.norm(b - orc.spmv((rp, col, val), host(xg))) <= 1e-10 * np.linalg.norm(b)


def _counting_context(g):
    """A context whose allocator notes the size of every buffer the library holds."""
    import torch
    ctx, sizes, device = g.Context(use_torch_allocator=False), {}, torch.cuda.current_device()

    def alloc(nbytes, stream, user):
        p = torch.cuda.caching_allocator_alloc(int(nbytes), device, stream or 0)
        sizes[p] = nbytes
        return p

    def dealloc(p, stream, user):
        del sizes[p]
        torch.cuda.caching_allocator_delete(p)

    ctx._cbs = (g.ALLOC_FN(alloc), g.DEALLOC_FN(dealloc))
    assert g._lib.gko_context_set_allocator(ctx.handle, ctx._cbs[0], ctx._cbs[1], None) == g.OK
    return ctx, sizes


@pytest.mark.parametrize("n,length,scattered,kept", [
    (299_999, 5, False, False),      # 1.5 million entries, from which on a matrix is searched for row patterns
    (300_001, 5, False, True),
    (700_001, 3, False, True),       # three entries a row
    (1_200_001, 2, False, False),    # two
    (60_001, 40, False, True),       # the longest rows with patterns
    (60_001, 41, False, False),
    (60_001, 30, True, False)])
def test_which_matrices_keep_row_patterns(g, n, length, scattered, kept):
    """A matrix whose rows are one list of column offsets keeps its patterns (a
    byte per row and the table) only where products gain from them; one of
    scattered columns has none."""
    import torch
    i = torch.arange(n, device="cuda")[:, None]
    j = torch.arange(length, device="cuda")
    m = 2 * n + length
    col = torch.sort(torch.randint(0, n // length, (n, length), device="cuda") * length, 1).values + j if scattered else i + j
    rp = torch.arange(n + 1, device="cuda", dtype=torch.int32) * length
    val = torch.ones(n * length, dtype=torch.float64, device="cuda")
    ctx, sizes = _counting_context(g)
    M = g.Matrix.from_csr(rp, col.reshape(-1).int(), val, n_cols=m, ctx=ctx)
    extra = sum(sizes.values()) - 4 * (n + 1) - 12 * n * length
    assert (extra >= n) if kept else extra == 0, extra
    M.close()
    assert not sizes


def test_creation_without_gain_from_patterns_is_not_searched(g):
    """Creating the 5-point matrix of 500 x 500, whose products gain nothing
    from row patterns, takes about as long as any matrix of its size."""
    import statistics
    import time

    import torch
    n = 250_000
    i = torch.arange(n, device="cuda")
    star = i[:, None] + torch.tensor([-500, -1, 0, 1, 500], device="cuda")
    other = torch.sort(torch.randint(0, n // 8, (n, 5), device="cuda") * 5, 1).values + torch.arange(5, device="cuda")
    ctx = g.Context()

    def seconds(col):
        ok = (col >= 0) & (col < n)
        rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(ok.sum(1), 0, out=rp[1:])
        rp, col = rp.int(), col[ok].int()
        val = torch.ones(col.numel(), dtype=torch.float64, device="cuda")
        times = []
        for _ in range(40):
            torch.cuda.synchronize()
            t = time.perf_counter()
            M = g.Matrix.from_csr(rp, col, val, ctx=ctx)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
            M.close()
        return statistics.median(times)

    seconds(star)
    a, b = seconds(star), seconds(other)
    assert a <= 1.4 * b, (a, b)


def _uneven_rows(lists, length, n):
    """As _pattern_rows, with lists from one entry to `length`, most of them short."""
    rng = np.random.default_rng(lists)
    spread = 2 * length + 40
    sizes = np.maximum(1, (length * rng.uniform(0, 1, lists) ** 2).astype(int))
    sizes[0], sizes[1] = length, 1
    pat = rng.integers(0, lists, n)
    pat[:lists] = np.arange(lists)
    padded = np.zeros((lists, length), np.int64)
    for k, l in enumerate(sizes):
        padded[k, :l] = np.sort(rng.choice(np.arange(-spread, spread), size=l, replace=False))
    lens = sizes[pat]
    inside = np.arange(length)[None, :] < lens[:, None]
    col = ((np.arange(n) + spread)[:, None] + padded[pat])[inside]
    rp = np.concatenate([[0], np.cumsum(lens)])
    return n, n + 2 * spread, rp.astype(np.int32), col.astype(np.int32)


@pytest.mark.parametrize("name", ["1x5x400001", "27x7x350063", "3x9x300064", "30x13x150001", "35x28x90001",
                                  "27x27x90001odd", "126x6x400000odd", "127x6x400000odd", "128x4x700001",
                                  "22x40x60001", "8x12x400001u", "30x13x400001u", "20x40x160001u", "24x32x200064u"])
def test_repeated_rows_above_the_search_limit(g, name):
    """As test_repeated_rows, with at least 1.5 million entries, and ("u") with
    rows of very different lengths, which end at different slots."""
    uneven = name.endswith("u")
    if uneven:
        n, m, rp, col = _uneven_rows(*(int(v) for v in name[:-1].split("x")))
    else:
        n, m, rp, col = _pattern_rows(name)
    assert len(col) >= 1_500_000
    rng = np.random.default_rng(6)
    val, lens = rng.uniform(-1, 1, len(col)), np.diff(rp)
    x, y0 = rng.uniform(-1, 1, m), rng.uniform(-1, 1, n)
    for f32 in (False, True):
        t = np.float32 if f32 else np.float64
        A = make(g, (n, m, rp, col, val.astype(t)), f32)
        xs, ys, vs = (v.astype(t).astype(np.float64) for v in (x, y0, val))
        terms = np.append(vs * xs[col], 0.0).astype(np.longdouble)
        want, size = (np.where(lens > 0, np.add.reduceat(v, rp[:-1]), 0.0) for v in (terms, np.abs(terms)))
        want, size = (1.5 * want + 0.5 * ys).astype(np.float64), (1.5 * size + 0.5 * np.abs(ys)).astype(np.float64)
        for fmt in ("csr", "ell", "sellp", "hybrid"):
            if uneven and fmt == "ell" and ell_infeasible((n, m, rp, col, val.astype(t)), 4 if f32 else 8):
                continue
            C = A.clone().convert(fmt)
            y = dev(y0.astype(t))
            g.spmv(C, 1.5, dev(x.astype(t)), 0.5, y)
            assert_spmv_close(host(y), want, size, lens, f32, "%s %s" % (name, fmt))
            C.close()
        A.close()


def _seconds(f, reps=20):
    import torch
    for _ in range(3):
        f()
    best = float("inf")
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / reps * 1e-3)
    return best


def test_ell_rows_end_at_their_padding(g):
    """ELL with row patterns, 28 slots a row for rows of 7 entries (one of 4096
    has 28): the FP32 product, too, stops where a wavefront's rows have ended,
    as seen from its time, which is below the FP64 product's (reading all
    slots, it took 1.2 times as long)."""
    import torch
    n = 2_000_003
    i = torch.arange(n, device="cuda")
    lens = torch.where(i % 4096 == 0, 28, 7)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=rp[1:])
    row = torch.repeat_interleave(i, lens)
    col = (row + torch.arange(row.numel(), device="cuda") - rp[row]).int()
    times = []
    for dt in (torch.float32, torch.float64):
        A = g.Matrix.from_csr(rp.int(), col, torch.ones(col.numel(), dtype=dt, device="cuda"), n_cols=n + 28)
        A.convert("ell")
        x, y = torch.ones(n + 28, dtype=dt, device="cuda"), torch.empty(n, dtype=dt, device="cuda")
        times.append(_seconds(lambda: g.spmv(A, 1.0, x, 0.0, y)))
        assert torch.equal(y, lens.to(dt))
        A.close()
    assert times[0] <= 0.9 * times[1], times


@pytest.mark.parametrize("length", [12, 16])
def test_fp32_rows_that_share_lds_banks(g, length):
    """FP32 rows of 12 and of 16 entries with row patterns: the CSR product is
    no slower than that of the same matrix with one column moved to where it
    has none (it took 1.05 and 1.13 times as long)."""
    import torch
    n = 24_000_000 // length
    rp = torch.arange(n + 1, device="cuda", dtype=torch.int32) * length
    col = (torch.arange(n, device="cuda")[:, None] + torch.arange(length, device="cuda")).int()
    val = torch.ones(n * length, dtype=torch.float32, device="cuda")
    x, y = torch.ones(n + length + 200, device="cuda"), torch.empty(n, device="cuda")
    other = col.clone()
    i = torch.arange(200, device="cuda")
    other[i, -1] = (i + length + i // 2).int()                # 200 lists of offsets: more than a table takes
    times = []
    for c in (col, other):
        A = g.Matrix.from_csr(rp, c.reshape(-1), val, n_cols=n + length + 200)
        times.append(min(_seconds(lambda: g.spmv(A, 1.0, x, 0.0, y)) for _ in range(2)))
        assert bool((y == length).all())
        A.close()
    assert times[0] <= 1.03 * times[1], times


@pytest.mark.parametrize("name", ["even64x72", "even64x73", "even63x95", "even65x96", "even130x97", "even3x2500",
                                  "even200x129", "even1x9000"])
@pytest.mark.parametrize("f32", [False, True])
def test_conversions_of_wide_tiles(g, orc, name, f32):
    """Rows on both sides of 72 slots, from which on a tile is converted in
    blocks of 64 rows and 32 slots, at the blocks' edges."""
    test_conversions_at_tile_and_chunk_edges(g, orc, name, f32)


@pytest.mark.parametrize("n,longest", [(64, 200), (333, 300), (2000, 120), (129, 3000)])
@pytest.mark.parametrize("f32", [False, True])
def test_conversions_of_uneven_wide_tiles(g, orc, n, longest, f32):
    """Rows of any length up to `longest`, the longest first: wide tiles beside
    narrow ones in SELL-P, tails behind wide tiles in HYB."""
    rng = np.random.default_rng(n)
    lens = np.sort((longest * rng.uniform(0, 1, n) ** 1.5).astype(int))[::-1]
    lens[0] = longest
    m = longest + 500
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(m, size=l, replace=False)) for l in lens]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(col)).astype(np.float32 if f32 else np.float64)
    A = make(g, (n, m, rp, col, vals.astype(np.float64)), f32)
    Ah = (rp, col, vals.astype(np.float64))
    s = A.convert("sellp").export_sellp()
    w, sets, sc, sv = orc.csr_to_sellp(Ah)
    assert np.array_equal(host(s["widths"]), w) and np.array_equal(host(s["sets"]), sets)
    assert np.array_equal(host(s["col"]), sc) and np.array_equal(bits(host(s["val"])), bits(sv.astype(vals.dtype)))
    s = A.convert("hybrid").export_storage()
    K, ld, ec, ev, tr, tc, tv = orc.csr_to_hyb(Ah, value_bytes=4 if f32 else 8)
    for key, want in (("ell_col", ec), ("coo_row", tr), ("coo_col", tc)):
        assert np.array_equal(host(s[key]), want), key
    for key, want in (("ell_val", ev), ("coo_val", tv)):
        assert np.array_equal(bits(host(s[key])), bits(want.astype(vals.dtype))), key
    s = A.convert("ell").export_storage()
    assert np.array_equal(host(s["ell_col"]), orc.csr_to_ell(Ah)[2])
    for fmt in ("ell", "sellp", "hybrid"):
        erp, ecol, evl = (host(t) for t in A.convert(fmt).convert("csr").export_csr())
        assert np.array_equal(erp, rp) and np.array_equal(ecol, col) and np.array_equal(bits(evl), bits(vals)), fmt


def test_conversion_time_does_not_grow_with_the_rows(g):
    """16 million entries take about as long to and from ELL in rows of 3,000 as
    in rows of 32 (they took 60 and 230 times as long)."""
    import time

    import torch
    best = {}
    for length in (32, 3000):
        n = 16_000_000 // length
        rp = torch.arange(n + 1, device="cuda", dtype=torch.int32) * length
        col = (torch.arange(n, device="cuda")[:, None] + torch.arange(length, device="cuda")).int().reshape(-1)
        A = g.Matrix.from_csr(rp, col, torch.ones(n * length, dtype=torch.float64, device="cuda"), n_cols=n + length)
        best[length] = [float("inf")] * 2
        for _ in range(5):
            for k, fmt in enumerate(("ell", "csr")):
                torch.cuda.synchronize()
                t = time.perf_counter()
                A.convert(fmt)
                torch.cuda.synchronize()
                best[length][k] = min(best[length][k], time.perf_counter() - t)
        A.close()
    assert all(b <= 3 * a for a, b in zip(best[32], best[3000])), best
