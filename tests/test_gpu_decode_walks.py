"""Decoding to CSR in two walks over eight segments (32 nonzeros of a lane) at
a time: lane lengths around that edge, escapes of columns and values, rows
that cross lanes and empty rows.  Columns and value bits are exact."""
import numpy as np
import pytest

import paper_2603_01915_amd as P
from gpu_common import need_gpu, progress

pytestmark = pytest.mark.gpu


def matrix(lens, n, dtype, escapes):
    rng = np.random.default_rng(len(lens) + n)
    rp = np.zeros(len(lens) + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    step = n // 128  # a column drawn from each of L strips of the row
    ci = np.concatenate([np.arange(L) * step + rng.integers(0, step, size=L) for L in lens]).astype(np.int32)
    if escapes:  # more symbols than table slots: both alphabets escape
        v = rng.standard_normal(len(ci)).astype(dtype)
    else:
        v = rng.choice([0.5, -1.5, 2.0], size=len(ci)).astype(dtype)
    return rp, ci, v


@pytest.mark.parametrize("layout,T", [("row", 0), ("nnz", 28), ("nnz", 32), ("nnz", 36), ("nnz", 100)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("escapes", [False, True])
@pytest.mark.parametrize("max_mult", [255, 256])
def test_two_walks(layout, T, dtype, escapes, max_mult):
    need_gpu()
    n = 1 << 22 if escapes else 640
    rng = np.random.default_rng(3)
    for lens in ([0, 1, 2, 3, 4, 5, 27, 28, 29, 31, 32, 33, 34, 35, 36, 63, 64, 65, 100], [32] * 64, [33] * 65,
                 list(rng.integers(0, 70, size=300))):
        progress("decode walks %s T=%d %s %d rows" % (layout, T, dtype.__name__, len(lens)))
        rp, ci, v = matrix(lens, n, dtype, escapes)
        A = P.Matrix.from_csr(rp, ci, v, n, layout=layout, lane_nnz=T, max_mult=max_mult)
        if escapes and len(ci) > 4500:
            info = A.info()
            assert info["esc_delta"] > 0 and info["esc_value"] > 0
        r2, c2, v2 = A.decode_csr()
        assert np.array_equal(r2.cpu().numpy(), rp) and np.array_equal(c2.cpu().numpy(), ci)
        assert np.array_equal(v2.cpu().numpy().view(np.uint8), v.view(np.uint8))


@pytest.mark.parametrize("dtype,short,long", [(np.float64, 7, 9), (np.float32, 15, 17)])
@pytest.mark.parametrize("shape", [(0, 0), (1, 1), (4, 2), (16, 1), (16, 2)])
def test_rows_by_groups(dtype, short, long, shape):
    """Rows dealt to groups of lanes: from four waves a CU and a mean row whose
    values fill 64 bytes (a little below and above that mean), row lengths
    around the walks' eight segments in one matrix, launch shapes of the
    caller's, a last wave of five rows."""
    torch = need_gpu()
    waves = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    for mean, rows in ((short, 64 * waves), (long, 64 * waves), (long, 64 * (waves - 1) + 5), (long, 64 * waves + 5)):
        lens = np.full(rows, mean)
        lens[:64 * 19] = np.repeat([0, 1, 2, 3, 4, 5, 27, 28, 29, 31, 32, 33, 34, 35, 36, 63, 64, 65, 100], 64)
        lens[:64] = np.arange(64)
        progress("rows by groups %s mean %d, %d rows, shape %s" % (dtype.__name__, mean, rows, shape))
        rp = np.zeros(rows + 1, np.int64)
        rp[1:] = np.cumsum(lens)
        within = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
        ci = (np.repeat(np.arange(rows), lens) + 2 * within).astype(np.int32)
        v = np.array([0.5, -1.5, 2.0, 0.25], dtype)[within % 4]
        rp, n = rp.astype(np.int32), rows + 200
        A = P.Matrix.from_csr(rp, ci, v, n, layout="row")
        assert A.info()["esc_delta"] == 0 and A.info()["esc_value"] == 0
        A.set_launch(*shape)
        r2, c2, v2 = A.decode_csr()
        assert np.array_equal(r2.cpu().numpy(), rp) and np.array_equal(c2.cpu().numpy(), ci)
        assert np.array_equal(v2.cpu().numpy().view(np.uint8), v.view(np.uint8))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("escapes", [False, True])
@pytest.mark.parametrize("max_mult", [255, 256])
@pytest.mark.parametrize("longest", [256, 257, 5001])
def test_lone_rows(dtype, escapes, max_mult, longest):
    """One row that takes longer than all the others (one walk instead of two):
    64 times a mean below four (256: not yet), and far beyond; short and empty
    rows around it."""
    need_gpu()
    lens = np.tile([0, 1, 2, 3, 5], 1400)
    lens[3001] = longest
    progress("decode lone row %d %s" % (longest, dtype.__name__))
    rp = np.zeros(len(lens) + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    rng = np.random.default_rng(longest)
    n = 6000 if not escapes else 1 << 20
    ci = np.concatenate([np.sort(rng.choice(n, size=L, replace=False)) for L in lens]).astype(np.int32)
    v = rng.standard_normal(len(ci)).astype(dtype) if escapes else rng.choice([0.5, 2.0], size=len(ci)).astype(dtype)
    A = P.Matrix.from_csr(rp, ci, v, n, layout="row", max_mult=max_mult)
    r2, c2, v2 = A.decode_csr()
    assert np.array_equal(r2.cpu().numpy(), rp) and np.array_equal(c2.cpu().numpy(), ci)
    assert np.array_equal(v2.cpu().numpy().view(np.uint8), v.view(np.uint8))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("longest,sort", [(40, 0), (400, 0), (400, 256)])
def test_unequal_rows_many_waves(dtype, longest, sort):
    """More waves than two walks keep resident, with short and with long chains
    (one walk); a last wave of five rows; rows in CSR order and sorted."""
    torch = need_gpu()
    rows = 64 * 16 * torch.cuda.get_device_properties(0).multi_processor_count + 69
    rng = np.random.default_rng(longest)
    lens = rng.integers(0, 6, size=rows)
    lens[rng.integers(0, rows, size=rows // 50)] = longest
    progress("decode unequal rows, longest %d %s sort %d" % (longest, dtype.__name__, sort))
    rp = np.zeros(rows + 1, np.int64)
    rp[1:] = np.cumsum(lens)
    within = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
    ci = (np.repeat(rng.integers(0, 5000, size=rows), lens) + 3 * within).astype(np.int32)
    v = rng.standard_normal(100).astype(dtype)[rng.integers(0, 100, size=len(ci))]
    rp = rp.astype(np.int32)
    A = P.Matrix.from_csr(rp, ci, v, 5000 + 3 * longest, layout="row", sort_window=sort)
    r2, c2, v2 = A.decode_csr()
    assert np.array_equal(r2.cpu().numpy(), rp) and np.array_equal(c2.cpu().numpy(), ci)
    assert np.array_equal(v2.cpu().numpy().view(np.uint8), v.view(np.uint8))
