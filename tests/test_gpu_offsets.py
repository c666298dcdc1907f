"""The largest entry count, 2^31 - 2: products and conversions whose last
entries lie within a step of the end of int32 (about 80 GB of device memory)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2011_08879_amd as g
    return g


@pytest.mark.parametrize("width,formats", [(64, ("csr", "coo", "ell")), (128, ("csr",))])
def test_largest_entry_count(g, width, formats):
    """Rows of `width` consecutive columns, the last one two entries short, and
    five empty rows behind it (64 entries: the kernels that stage entries
    through LDS; 128: the subwarp per row).  Whole numbers, so the sums are
    exact: the difference of two entries of x's running sum."""
    import torch
    nnz = 2 ** 31 - 2
    full = 2 ** 31 // width
    n = full + 5
    rp = torch.arange(n + 1, dtype=torch.int64, device="cuda").mul_(width).clamp_(max=nnz).to(torch.int32)
    col = torch.arange(nnz, dtype=torch.int32, device="cuda")
    start = col.div(width, rounding_mode="floor").clamp_(max=n - width)
    col.remainder_(width).add_(start)
    del start
    x = torch.arange(n, device="cuda").remainder_(7).float()
    run = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(x.long(), 0, out=run[1:])
    c0 = torch.arange(n, device="cuda").clamp_(max=n - width)
    lens = (rp[1:] - rp[:-1]).long()
    want = (run[c0 + lens] - run[c0]).float()
    ctx = g.Context()
    A = g.Matrix.from_csr(rp, col, torch.ones(nnz, dtype=torch.float32, device="cuda"), ctx=ctx)
    for fmt in formats:
        A.convert(fmt)
        y = torch.full((n,), -1.0, device="cuda")
        g.spmv(A, 1.0, x, 0.0, y)
        assert torch.equal(y, want), fmt
        erp, ecol, ev = A.export_csr()
        assert torch.equal(erp, rp) and torch.equal(ecol, col) and bool((ev == 1).all()), fmt
        del erp, ecol, ev
        torch.cuda.empty_cache()
    A.close()
    del A, rp, col
    torch.cuda.empty_cache()
