"""The symmetric product's block sums in LDS: more blocks of y than LDS holds
(elements that go to y directly), an order that is no multiple of a block,
several rounds of waves, and every table format, against the oracle."""
import numpy as np
import pytest
import scipy.sparse as sp

import paper_2603_01915_amd as P
import workloads
from gpu_common import check_spmv, need_gpu, progress

pytestmark = pytest.mark.gpu


def symmetric(n, per_row, band, dtype):
    rng = np.random.default_rng(n + band)
    r = np.repeat(np.arange(n), per_row)
    c = np.clip(r + rng.integers(1, band + 1, size=len(r)), 0, n - 1)
    keep = c > r
    U = sp.csr_matrix((rng.choice([0.5, -1.5, 2.0], size=int(keep.sum())), (r[keep], c[keep])), shape=(n, n))
    U.sum_duplicates()
    A = (U + U.T + sp.diags(rng.standard_normal(n))).tocsr()
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data.astype(dtype)


# 64 elements a block, 128 blocks: one below, at and past what LDS holds; far
# columns past the windows; a single row beyond a block
@pytest.mark.parametrize("n,band", [(63, 5), (65, 64), (8192, 300), (8193, 8193), (20011, 20011), (150001, 40)])
@pytest.mark.parametrize("layout,T", [("row", 0), ("nnz", 16)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("options", [{}, {"max_mult": 256}, {"escape_in_stream": True}])
def test_block_sums(n, band, layout, T, dtype, options):
    torch = need_gpu()
    rp, ci, v = symmetric(n, 6, band, dtype)
    rpu, ciu, vu, d = P.symmetric_split(rp, ci, v)
    progress("sym blocks n=%d band=%d %s %s %s" % (n, band, layout, dtype.__name__, options))
    M = P.Matrix.from_csr(rpu, ciu, vu, n, layout=layout, lane_nnz=T, **options)
    x, y0 = workloads.vector(n, 3, dtype), workloads.vector(n, 4, dtype)
    y = torch.from_numpy(y0.copy()).cuda()
    M.spmv_sym(torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda(), y, alpha=-0.5, beta=0.75)
    check_spmv(y.cpu().numpy(), rp, ci, v, x, y0, -0.5, 0.75, dtype)
