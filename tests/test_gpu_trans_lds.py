"""The transposed product with dX privatised in LDS: one and two column
blocks, the widths of its passes, more passes than one launch takes, and
columns of A a multiple of 32 apart, against the oracle.

Tolerances: the sums in LDS are FP64; an FP32 result rounds each workgroup's
copy and then the sum of the copies once, 2 * 2^-24 of |A^T||dY| at most."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import paper_2603_01915_amd as P
import workloads
from gpu_common import need_gpu, progress, rel_error

pytestmark = pytest.mark.gpu
TOLERANCE = {np.float64: 1e-12, np.float32: 3 * 2.0 ** -24}
ROOM = {np.float64: (160 - 80) * 1024 // 8, np.float32: (160 - 64) * 1024 // 8}  # FP64 elements of the block


def matrix(m, n, dtype, step=1):
    rng = np.random.default_rng(n + 7 * m)
    lens = np.minimum(rng.integers(0, 60, size=m), (n + step - 1) // step)
    rp = np.zeros(m + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    top = (n + step - 1) // step
    ci = np.concatenate([np.sort(rng.choice(top, size=L, replace=False)) * step for L in lens] +
                        [np.zeros(0, np.int64)]).astype(np.int32)
    v = rng.choice([0.5, -1.5, 2.0, 0.25], size=len(ci)).astype(dtype)
    return rp, ci, v


def check(torch, rp, ci, v, n, k, dtype, layout, T):
    m = len(rp) - 1
    A = P.Matrix.from_csr(rp, ci, v, n, layout=layout, lane_nnz=T)
    ld = k + 3
    dY = np.full((m, ld), np.nan, dtype)  # columns past k must not be read
    dY[:, :k] = workloads.vector(m, 6, dtype, k=k)
    dX0 = workloads.vector(n, 3, dtype, k=ld)
    dX = torch.from_numpy(dX0.copy()).cuda()
    A.spmm_t(torch.from_numpy(dY).cuda()[:, :k], dX[:, :k], alpha=-0.75, beta=0.5)
    out = dX.cpu().numpy()
    assert np.array_equal(out[:, k:], dX0[:, k:])
    At = sp.csr_matrix((v.astype(np.float64), ci, rp), shape=(m, n)).T.tocsr()
    At.sort_indices()
    for c in range(k):
        y = np.ascontiguousarray(dY[:, c])
        ref = oracle.spmtv(rp, ci, v, n, y, np.ascontiguousarray(dX0[:, c]), alpha=-0.75, beta=0.5)
        scale = 0.75 * oracle.absmv(At.indptr, At.indices, At.data, y) + 0.5 * np.abs(dX0[:, c].astype(np.float64))
        assert rel_error(out[:, c], ref, scale) <= TOLERANCE[dtype], (n, k, c)


@pytest.mark.parametrize("layout,T", [("row", 0), ("nnz", 32)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_block_edges(layout, T, dtype):
    torch = need_gpu()
    room = ROOM[dtype]
    # a whole block, one column more, two whole blocks, one more (global
    # atomics), and a single column
    for n in (room, room + 1, 2 * room, 2 * room + 1, 1):
        progress("trans block n=%d %s %s" % (n, layout, dtype.__name__))
        check(torch, *matrix(700, n, dtype), n, 2, dtype, layout, T)


@pytest.mark.parametrize("layout,T", [("row", 0), ("nnz", 32)])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 7, 8, 9, 100])
def test_pass_widths(layout, T, k):
    torch = need_gpu()
    # 4096 columns: three a pass (100: 34 passes, more than one launch); 300: eight
    for n in (4096, 300):
        progress("trans width n=%d k=%d %s" % (n, k, layout))
        check(torch, *matrix(500, n, np.float32), n, k, np.float32, layout, T)


def test_columns_32_apart():
    torch = need_gpu()
    check(torch, *matrix(900, 4096, np.float64, step=32), 4096, 2, np.float64, "nnz", 32)


@pytest.mark.parametrize("layout,T", [("row", 0), ("nnz", 32)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_limit_of_the_blocks(layout, T, dtype):
    """The longest dX that two column blocks hold, and one column more (global
    atomic adds, in column chunks of 4 and 1)."""
    torch = need_gpu()
    for n in (2 * ROOM[dtype], 2 * ROOM[dtype] + 1):
        progress("trans limit n=%d %s %s" % (n, layout, dtype.__name__))
        check(torch, *matrix(1500, n, dtype), n, 5, dtype, layout, T)


@pytest.mark.parametrize("layout,T", [("row", 0), ("nnz", 32)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_waves_dealt_in_turn(layout, T, dtype):
    """Encoded waves around the number of workgroups and of wavefronts a pass
    has: one, fewer than a workgroup's 16, no multiple of either, and more
    than one round of every wavefront."""
    torch = need_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for rows in (1, 64 * 5, 64 * 33 + 1, 64 * 130):
        progress("trans waves %d rows %s %s" % (rows, layout, dtype.__name__))
        check(torch, *matrix(rows, 257, dtype), 257, 3, dtype, layout, T)
    # one nonzero a row: 17 waves for every wavefront of a CU's workgroup
    m, n = 64 * (16 * cus + 1) + 3, 97
    rp, ci = np.arange(m + 1, dtype=np.int32), (np.arange(m) * 31 % n).astype(np.int32)
    check(torch, rp, ci, np.full(m, 0.5, dtype), n, 1, dtype, layout, T)
