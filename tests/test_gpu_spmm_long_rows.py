"""Products with 32 FP32 columns and the variant for long rows: from 2^24
nonzeros and a mean row of 1024 in the nonzero layout, and just below either
bound; row ends at the ends of lanes and inside them, empty rows, a last lane
that is not full, more than 32 columns, both table formats."""
import numpy as np
import pytest

import oracle
import paper_2603_01915_amd as P
import workloads
from gpu_common import TOL, need_gpu, progress, rel_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,mean,T", [(16384, 1024, 0), (16384, 1023, 0), (8195, 2051, 60), (8195, 2051, 44)])
@pytest.mark.parametrize("k,options", [(32, {}), (37, {"max_mult": 256})])
def test_long_rows(rows, mean, T, k, options):
    torch = need_gpu()
    n = 6000
    rng = np.random.default_rng(rows + mean)
    lens = np.full(rows, mean)
    # (rows in pairs that keep the mean: lengths around lanes, empty rows)
    lens[0:200:2] = rng.integers(0, 130, size=100)
    lens[200], lens[202], lens[204] = 0, 0, 1
    lens[1:206:2] += mean - lens[0:205:2]
    rp = np.zeros(rows + 1, np.int64)
    rp[1:] = np.cumsum(lens)
    assert rp[-1] == rows * mean
    within = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
    start = np.repeat(rng.integers(0, n - lens.max(), size=rows), lens)
    ci = (start + within).astype(np.int32)
    v = rng.standard_normal(64).astype(np.float32)[rng.integers(0, 64, size=len(ci))]
    rp = rp.astype(np.int32)
    progress("spmm long rows %d of %d T=%d k=%d" % (rows, mean, T, k))
    A = P.Matrix.from_csr(rp, ci, v, n, layout="nnz", lane_nnz=T, **options)
    X, Y0 = workloads.vector(n, 3, np.float32, k=k), workloads.vector(rows, 4, np.float32, k=k)
    ld = (k + 3) // 4 * 4
    Xd = torch.zeros((n, ld), dtype=torch.float32, device="cuda")
    Xd[:, :k] = torch.from_numpy(X)
    Y = torch.from_numpy(Y0.copy()).cuda()
    A.spmm(Xd[:, :k], Y, alpha=-0.5, beta=0.75)
    Y = Y.cpu().numpy()
    for c in (0, 1, 13, 31, k - 1):
        x = np.ascontiguousarray(X[:, c])
        ref = oracle.spmv(rp, ci, v, x, np.ascontiguousarray(Y0[:, c]), alpha=-0.5, beta=0.75)
        scale = 0.5 * oracle.absmv(rp, ci, v, x) + 0.75 * np.abs(Y0[:, c].astype(np.float64))
        assert rel_error(Y[:, c], ref, scale) <= TOL[np.float32], (c,)
