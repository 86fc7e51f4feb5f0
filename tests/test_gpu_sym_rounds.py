"""The symmetric product over several rounds of waves: sums flushed between
rounds, blocks claimed anew, an odd number of rounds, in both layouts and
under launch shapes of the caller's, against the oracle."""
import numpy as np
import pytest

import paper_2603_01915_amd as P
import workloads
from gpu_common import check_spmv, need_gpu, progress
from test_gpu_sym_blocks import symmetric

pytestmark = pytest.mark.gpu


def check(torch, M, rp, ci, v, d, dtype):
    n = len(rp) - 1
    x, y0 = workloads.vector(n, 3, dtype), workloads.vector(n, 4, dtype)
    y = torch.from_numpy(y0.copy()).cuda()
    M.spmv_sym(torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda(), y, alpha=-0.5, beta=0.75)
    check_spmv(y.cpu().numpy(), rp, ci, v, x, y0, -0.5, 0.75, dtype)


@pytest.mark.parametrize("band", [40, 200000])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_three_rounds(band, dtype):
    """33 or more encoded waves to a workgroup of 16 wavefronts."""
    torch = need_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 64 * 33 * cus + 17
    rp, ci, v = symmetric(n, 5, band, dtype)
    rpu, ciu, vu, d = P.symmetric_split(rp, ci, v)
    for layout, T in (("row", 0), ("nnz", 4)):
        progress("sym rounds n=%d band=%d %s %s" % (n, band, layout, dtype.__name__))
        M = P.Matrix.from_csr(rpu, ciu, vu, n, layout=layout, lane_nnz=T)
        assert M.info()["num_waves"] > 32 * cus
        check(torch, M, rp, ci, v, d, dtype)


@pytest.mark.parametrize("shape", [(1, 1), (2, 1), (3, 2), (4, 1), (4, 4), (16, 1), (16, 2), (12, 2)])
@pytest.mark.parametrize("layout,T", [("row", 0), ("nnz", 8)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_launch_shapes(shape, layout, T, dtype):
    torch = need_gpu()
    n = 100003  # with one wavefront a CU: seven rounds in the row layout
    rp, ci, v = symmetric(n, 5, 900, dtype)
    rpu, ciu, vu, d = P.symmetric_split(rp, ci, v)
    progress("sym shape %s %s %s" % (shape, layout, dtype.__name__))
    M = P.Matrix.from_csr(rpu, ciu, vu, n, layout=layout, lane_nnz=T)
    M.set_launch(*shape)
    check(torch, M, rp, ci, v, d, dtype)
