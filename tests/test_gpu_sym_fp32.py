"""The FP32 symmetric product sums in FP64 and rounds y once: random matrices
(elements with and without a block in LDS), a band, and a dense first row and
last column (sums of many flushes), in both layouts.

Tolerance: products of two FP32 numbers are exact in FP64, so y differs from
the oracle's FP64 result by one rounding, 2^-24 of |y|, and by the rounding of
the two FP64 sums: one per term of a row, less than 2 * 2^-53 * 2^15 of
|alpha| |A| |x| + |beta| |y0| for up to 2^15 terms."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import paper_2603_01915_amd as P
import workloads
from gpu_common import need_gpu, progress

pytestmark = pytest.mark.gpu


def random_upper(n, per_row, band):
    rng = np.random.default_rng(n + band)
    r = np.repeat(np.arange(n), per_row)
    c = r + rng.integers(1, band + 1, size=len(r))
    keep = c < n
    return r[keep], c[keep]


def arrow_upper(n, per_row, band):
    r, c = random_upper(n, per_row, band)
    i = np.arange(n)
    return np.concatenate([r, np.zeros(n - 1, np.int64), i[:-1]]), np.concatenate([c, i[1:], np.full(n - 1, n - 1)])


@pytest.mark.parametrize("make,n,per_row,band", [
    (random_upper, 300, 5, 300), (random_upper, 4000, 12, 4000), (random_upper, 20000, 12, 20000),
    (random_upper, 30011, 6, 30011), (random_upper, 30011, 12, 50), (arrow_upper, 30011, 3, 200)])
@pytest.mark.parametrize("layout,T", [("row", 0), ("nnz", 16)])
@pytest.mark.parametrize("with_diag", [True, False])
def test_one_rounding(make, n, per_row, band, layout, T, with_diag):
    torch = need_gpu()
    r, c = make(n, per_row, band)
    rng = np.random.default_rng(9)
    U = sp.csr_matrix((np.ones(len(r)), (r, c)), shape=(n, n))
    U.sum_duplicates()
    U.sort_indices()
    v = rng.standard_normal(200).astype(np.float32)[rng.integers(0, 200, size=U.nnz)]
    d = rng.standard_normal(n).astype(np.float32) if with_diag else np.zeros(n, np.float32)
    progress("sym fp32 %s n=%d band=%d %s" % (make.__name__, n, band, layout))
    M = P.Matrix.from_csr(U.indptr.astype(np.int32), U.indices.astype(np.int32), v, n, layout=layout, lane_nnz=T)
    x, y0 = workloads.vector(n, 3, np.float32), workloads.vector(n, 4, np.float32)
    y = torch.from_numpy(y0.copy()).cuda()
    M.spmv_sym(torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda() if with_diag else None, y, alpha=-0.5, beta=0.75)
    S = sp.csr_matrix((v.astype(np.float64), U.indices, U.indptr), shape=(n, n))
    A = (S + S.T + sp.diags(d.astype(np.float64))).tocsr()
    A.sort_indices()
    rp, ci = A.indptr.astype(np.int32), A.indices.astype(np.int32)
    x64, y64 = x.astype(np.float64), y0.astype(np.float64)
    ref = oracle.spmv(rp, ci, A.data, x64, y64, alpha=-0.5, beta=0.75)
    scale = 0.5 * oracle.absmv(rp, ci, A.data, x64) + 0.75 * np.abs(y64)
    bound = 2.0 ** -24 * np.abs(ref) + 2.0 ** -37 * scale
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - ref) <= bound)


def test_no_nonzeros():
    torch = need_gpu()
    n = 70
    M = P.Matrix.from_csr(np.zeros(n + 1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32), n)
    x, y0, d = (workloads.vector(n, i, np.float32) for i in (3, 4, 5))
    y = torch.from_numpy(y0.copy()).cuda()
    M.spmv_sym(torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda(), y, alpha=2.0, beta=0.5)
    ref = 2.0 * d.astype(np.float64) * x + 0.5 * y0.astype(np.float64)
    assert np.all(np.abs(y.cpu().numpy() - ref) <= 2.0 ** -24 * np.abs(ref) + 2.0 ** -37 * (2 * np.abs(d * x) + np.abs(y0)))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_captured(dtype):
    """Replays of a captured product, with eager products of another vector and
    the handle's other products (which use the same scratch) between them."""
    torch = need_gpu()
    n = 5000
    r, c = random_upper(n, 7, 900)
    U = sp.csr_matrix((np.ones(len(r)), (r, c)), shape=(n, n))
    U.sum_duplicates()
    U.sort_indices()
    rng = np.random.default_rng(3)
    v = rng.standard_normal(200).astype(dtype)[rng.integers(0, 200, size=U.nnz)]
    progress("sym captured %s" % dtype.__name__)
    M = P.Matrix.from_csr(U.indptr.astype(np.int32), U.indices.astype(np.int32), v, n, layout="nnz", lane_nnz=16)
    M.to_device()
    x, other = (torch.from_numpy(workloads.vector(n, i, dtype)).cuda() for i in (3, 4))
    y = torch.zeros_like(x)
    M.spmv_sym(x, None, y)  # loads the kernels
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        M.spmv_sym(x, None, y)
    S = sp.csr_matrix((v.astype(np.float64), U.indices, U.indptr), shape=(n, n))
    A = (S + S.T).tocsr()
    A.sort_indices()
    rp, ci = A.indptr.astype(np.int32), A.indices.astype(np.int32)
    for i in range(4):
        x.copy_(torch.from_numpy(workloads.vector(n, 10 + i, dtype)))
        y.fill_(float("nan"))
        graph.replay()
        M.spmv_sym(other)
        M.spmm_t(other[:, None].contiguous())
        M.spmv(other)
        torch.cuda.synchronize()
        xs = x.cpu().numpy().astype(np.float64)
        ref = oracle.spmv(rp, ci, A.data, xs)
        unit = 2.0 ** -24 if dtype == np.float32 else 2.0 ** -53
        bound = unit * np.abs(ref) + (2.0 ** -37 if dtype == np.float32 else 1e-12) * oracle.absmv(rp, ci, A.data, xs)
        assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - ref) <= bound), i
