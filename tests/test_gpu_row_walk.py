"""The nonzero layout's row walk: segments that cross up to four rows (rows of
one nonzero), empty rows between them, rows ending at the ends of lanes and
waves, escapes inside them, and grids of fewer waves than wavefronts."""
import numpy as np
import pytest

import oracle
import paper_2603_01915_amd as P
import workloads
from gpu_common import TOL, check_spmv, need_gpu, progress, rel_error

pytestmark = pytest.mark.gpu


def matrix(lens, n, dtype, distinct):
    rng = np.random.default_rng(len(lens) + n + distinct)
    rp = np.zeros(len(lens) + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    step = max(1, n // 512)  # a column drawn from each of L strips of the row
    ci = np.concatenate([np.arange(L) * step + rng.integers(0, step, size=L) for L in lens]).astype(np.int32)
    v = rng.standard_normal(distinct).astype(dtype)[rng.integers(0, distinct, size=len(ci))]
    return rp, ci, v


LENGTHS = {
    "ones": [1] * 1000,
    "ones and empty": [1, 0, 0] * 500 + [0] * 7,
    "lane ends": [16, 15, 17, 1, 3, 4, 5, 8, 24, 0, 64, 2, 2, 2] * 40,
    "one wave": [16] * 64,
    "one wave and one nonzero": [16] * 64 + [1],
    "long among short": [1] * 70 + [500] + [1, 2, 3] * 50 + [0] * 5 + [333],
    "many": None,
}


@pytest.mark.parametrize("name", list(LENGTHS))
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("distinct,options", [(7, {}), (7, {"max_mult": 256}), (9000, {}),
                                              (9000, {"escape_in_stream": True})])
def test_row_walk(name, dtype, distinct, options):
    torch = need_gpu()
    lens = LENGTHS[name]
    if lens is None:  # more waves than one round of the device's wavefronts
        lens = np.random.default_rng(5).integers(0, 9, size=1_700_000)
    n = 600 if distinct < 100 else 1 << 20
    rp, ci, v = matrix(lens, n, dtype, distinct)
    progress("row walk %s %s %d %s" % (name, dtype.__name__, distinct, options))
    A = P.Matrix.from_csr(rp, ci, v, n, layout="nnz", lane_nnz=16, **options)
    x, y0 = workloads.vector(n, 3, dtype), workloads.vector(len(lens), 4, dtype)
    y = torch.from_numpy(y0.copy()).cuda()
    A.spmv(torch.from_numpy(x).cuda(), y, alpha=-0.5, beta=0.75)
    check_spmv(y.cpu().numpy(), rp, ci, v, x, y0, -0.5, 0.75, dtype)
    if len(lens) > 100000:
        return
    for k in (3, 8, 16):  # per-lane columns and lane groups
        X = workloads.vector(n, 5, dtype, k=k)
        Y = A.spmm(torch.from_numpy(X).cuda()).cpu().numpy()
        ref = oracle.spmm(rp, ci, v, X)
        for c in range(k):
            assert rel_error(Y[:, c], ref[:, c], oracle.absmv(rp, ci, v, np.ascontiguousarray(X[:, c]))) <= TOL[dtype]


@pytest.mark.parametrize("n", [1, 2, 4095, 4096, 4097])
@pytest.mark.parametrize("options", [{}, {"max_mult": 256}])
def test_x_in_lds(n, options):
    """Single FP32 vectors around the length that LDS holds beside the tables."""
    torch = need_gpu()
    progress("x in LDS n=%d %s" % (n, options))
    rng = np.random.default_rng(n)
    lens = np.minimum(rng.integers(0, 90, size=700), n)
    rp = np.zeros(701, np.int32)
    rp[1:] = np.cumsum(lens)
    ci = np.concatenate([np.sort(rng.choice(n, size=L, replace=False)) for L in lens]).astype(np.int32)
    v = rng.standard_normal(50).astype(np.float32)[rng.integers(0, 50, size=len(ci))]
    A = P.Matrix.from_csr(rp, ci, v, n, layout="nnz", lane_nnz=32, **options)
    x, y0 = workloads.vector(n, 3, np.float32), workloads.vector(700, 4, np.float32)
    y = torch.from_numpy(y0.copy()).cuda()
    A.spmv(torch.from_numpy(x).cuda(), y, alpha=1.5, beta=-0.25)
    check_spmv(y.cpu().numpy(), rp, ci, v, x, y0, 1.5, -0.25, np.float32)
