"""The work that is timed: dtANS-compressed sparse products on one GPU.

A case is one use of the package as a program makes it: the matrix is encoded
and on the device, the vectors are device tensors, and a pass is one product
(one training step, one decode, one encode with its first product).  Matrices
are made on the GPU from the seed, with the structure and values of the
synthetic inputs of ``workloads``: banded rows, 27-point stencils, R-MAT
graphs, rows of skewed length, pruned weights.
"""
from __future__ import annotations

import math

import torch

import paper_2603_01915_amd as P
from paper_2603_01915_amd.autograd import DtansLinear

DEV = "cuda"

# Compressed stream bits per nonzero that the encoder reaches on each kind of
# matrix (word and escape streams, without tables and index).
_BITS = {"band": 18.0, "stencil": 14.3, "rmat": 27.0, "skewed": 27.4, "pruned": 14.4, "sym": 19.7}


def listed():
    return [
        # the smallest call: one product with a small banded matrix, as inside
        # an iterative solver; launches and latency are all of it
        {"name": "band_4k_f64", "kind": "band", "m": 4096, "per_row": 16, "k": 1, "f64": True},
        # the benchmark's workload: a 27-point stencil on 128^3
        {"name": "stencil_128_f64", "kind": "stencil", "g": 128, "k": 1, "f64": True, "paper": False},
        # a power-law graph: irregular rows, escapes, random gathers
        {"name": "rmat_22_f32", "kind": "rmat", "scale": 22, "k": 1, "f64": False, "in_stream": False},
        # rows of skewed length, an odd number of them
        {"name": "skewed_1m_f64", "kind": "skewed", "m": 1000003, "k": 1, "f64": True},
        # a pruned weight in decoding with batch 1 ...
        {"name": "pruned_f32_k1", "kind": "pruned", "m": 11008, "n": 4096, "k": 1, "f64": False},
        # ... with a small batch ...
        {"name": "pruned_f32_k8", "kind": "pruned", "m": 11008, "n": 4096, "k": 8, "f64": False},
        # ... and with a larger one
        {"name": "pruned_f32_k32", "kind": "pruned", "m": 11008, "n": 4096, "k": 32, "f64": False},
        # a training step through the pruned weight, stored once: forward and
        # gradient of the input
        {"name": "train_f32_b16", "kind": "train", "m": 11008, "n": 4096, "k": 16, "f64": False},
        # many small matrices in one launch
        {"name": "batch_64_f32", "kind": "batch", "count": 64, "lo": 10, "hi": 16, "k": 1, "f64": False,
         "sort": False},
        # a symmetric stencil stored as one triangle
        {"name": "sym_96_f64", "kind": "sym", "g": 96, "k": 1, "f64": True},
        # back to CSR: every column and value of a stencil
        {"name": "decode_100_f64", "kind": "decode", "of": "stencil", "g": 100, "f64": True},
        # a weight encoded anew after pruning, from device arrays, and its
        # first product
        {"name": "encode_f32", "kind": "encode", "of": "pruned", "m": 5504, "n": 4096, "f64": False},
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["band", "stencil", "rmat", "skewed", "pruned", "pruned", "train", "batch", "sym", "decode",
                       "encode"])
    f64 = rng.random() < 0.5
    if kind == "band":
        return {"kind": kind, "m": log(1000, 65536), "per_row": rng.randint(4, 64), "k": rng.choice([1, 1, 2, 4, 7]),
                "f64": f64}
    if kind == "stencil":
        return {"kind": kind, "g": log(20, 128), "k": rng.choice([1, 1, 1, 2, 4]), "f64": f64,
                "paper": rng.random() < 0.25}
    if kind == "rmat":
        return {"kind": kind, "scale": rng.randint(15, 21), "k": 1, "f64": f64, "in_stream": rng.random() < 0.3}
    if kind == "skewed":
        return {"kind": kind, "m": log(20000, 1000000), "k": rng.choice([1, 1, 3]), "f64": f64}
    if kind in ("pruned", "train"):
        return {"kind": kind, "m": log(300, 11008), "n": log(256, 4096),
                "k": rng.choice([1, 2, 3, 4, 5, 8, 12, 16, 24, 32]), "f64": kind == "pruned" and rng.random() < 0.25}
    if kind == "batch":
        return {"kind": kind, "count": log(4, 64), "lo": 10, "hi": rng.randint(11, 15), "k": rng.choice([1, 1, 2, 8]),
                "f64": f64, "sort": rng.random() < 0.3}
    if kind == "sym":
        return {"kind": kind, "g": log(16, 96), "k": 1, "f64": f64}
    if rng.random() < 0.5:
        return {"kind": kind, "of": "stencil", "g": log(20, 90 if kind == "decode" else 40), "f64": f64}
    return {"kind": kind, "of": "pruned", "m": log(300, 5504), "n": log(256, 4096), "f64": False}


# ------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform(shape, dtype, gen):
    return torch.rand(shape, dtype=dtype, device=DEV, generator=gen) * 2 - 1


def _dtype(case):
    return torch.float64 if case["f64"] else torch.float32


def _csr(m, rows, cols, vals):
    """COO sorted by (row, column) -> CSR (row_ptr and columns int32)."""
    rp = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(rows, minlength=m), 0, out=rp[1:])
    return rp.to(torch.int32), cols.to(torch.int32), vals.contiguous()


def _pool_values(count, pool, dtype, gen):
    values = torch.randn(pool, dtype=dtype, device=DEV, generator=gen)
    return values[torch.randint(0, pool, (count,), device=DEV, generator=gen)]


def _near_diagonal(m, lengths, half, pool, dtype, gen):
    """Columns uniform within +-half of the diagonal, duplicates merged."""
    rows = torch.repeat_interleave(torch.arange(m, device=DEV), lengths)
    cols = rows + torch.randint(-half, half + 1, (rows.numel(),), device=DEV, generator=gen)
    key = torch.unique(rows * m + cols.clamp_(0, m - 1))
    return _csr(m, key // m, key % m, _pool_values(key.numel(), pool, dtype, gen))


def _stencil(g, dtype, gen, upper=False):
    """The 27-point stencil on a g^3 grid (`upper`: the strict upper triangle),
    a coefficient for each offset times a scale for the octant of the row."""
    coef = torch.randn(27, dtype=dtype, device=DEV, generator=gen)
    scale = torch.rand(8, dtype=dtype, device=DEV, generator=gen) * 1.5 + 0.5
    i = torch.arange(g ** 3, device=DEV)
    z, y, x = i // (g * g), i // g % g, i % g
    octant = (z >= g // 2) * 4 + (y >= g // 2) * 2 + (x >= g // 2)
    d = torch.arange(27, device=DEV)
    dz, dy, dx = d // 9 - 1, d // 3 % 3 - 1, d % 3 - 1
    keep = torch.ones((g ** 3, 27), dtype=torch.bool, device=DEV)
    for c, dc in ((z, dz), (y, dy), (x, dx)):
        n = c[:, None].to(torch.int16) + dc[None, :].to(torch.int16)
        keep &= (n >= 0) & (n < g)
    off = dz * g * g + dy * g + dx
    if upper:
        keep &= (off > 0)[None, :]
    at = keep.view(-1).nonzero().view(-1)
    rows, o = at // 27, at % 27
    return _csr(g ** 3, rows, rows + off[o], coef[o] * scale[octant[rows]])


def _rmat(scale, dtype, gen):
    n, want = 1 << scale, 16 << scale
    key = torch.zeros(want + want // 8, dtype=torch.int64, device=DEV)
    row = torch.zeros_like(key)
    for _ in range(scale):
        u = torch.rand(key.numel(), device=DEV, generator=gen)
        down, right = u >= 0.76, ((u >= 0.57) & (u < 0.76)) | (u >= 0.95)
        row = (row << 1) | down
        key = (key << 1) | right
    key = torch.unique((row << scale) | key)
    vals = torch.tensor([0.5, 1.0, 2.0], dtype=dtype, device=DEV)
    return _csr(n, key >> scale, key & (n - 1),
                vals[torch.randint(0, 3, (key.numel(),), device=DEV, generator=gen)])


def _pruned(m, n, dtype, gen):
    """N(0, 0.02^2) rounded to bfloat16, the larger half kept."""
    w = (torch.randn(m, n, device=DEV, generator=gen) * 0.02).to(torch.bfloat16).float()
    bar = torch.sort(w.abs().view(-1)).values[m * n // 2]
    keep = (w.abs() >= bar) & (w != 0)
    at = keep.nonzero()
    return _csr(m, at[:, 0], at[:, 1], w[keep].to(dtype))


def _matrix(case, kind, gen):
    """(row_ptr, columns, values, number of columns) of the case's matrix."""
    dtype = _dtype(case)
    if kind == "band":
        m = case["m"]
        lengths = torch.full((m,), case["per_row"], dtype=torch.int64, device=DEV)
        return *_near_diagonal(m, lengths, 256, 64, dtype, gen), m
    if kind == "stencil":
        return *_stencil(case["g"], dtype, gen), case["g"] ** 3
    if kind == "sym":
        return *_stencil(case["g"], dtype, gen, upper=True), case["g"] ** 3
    if kind == "rmat":
        return *_rmat(case["scale"], dtype, gen), 1 << case["scale"]
    if kind == "skewed":
        m = case["m"]
        u = torch.rand(m, dtype=torch.float64, device=DEV, generator=gen)
        lomax = (1 - u) ** (-1 / 1.3) - 1
        lengths = (1 + torch.floor(6 * lomax)).clamp_(max=512).to(torch.int64)
        return *_near_diagonal(m, lengths, 32768, 256, dtype, gen), m
    return *_pruned(case["m"], case["n"], dtype, gen), case["n"]


def _batch_sizes(case):
    """Rows of the matrices of a batch: powers of two spread evenly."""
    span = case["hi"] - case["lo"]
    return [int(round(2 ** (case["lo"] + span * ((i * 0.61803398875) % 1)))) for i in range(case["count"])]


def _inputs(case, seed):
    """The case's matrices and vectors."""
    gen, kind, dtype = _gen(seed), case["kind"], _dtype(case)
    if kind == "batch":
        mats, xs = [], []
        for m in _batch_sizes(case):
            lengths = torch.randint(8, 65, (m,), device=DEV, generator=gen)
            mats.append((*_near_diagonal(m, lengths, 512, 64, dtype, gen), m))
            xs.append(_uniform((m,) if case["k"] == 1 else (m, case["k"]), dtype, gen))
        return {"mats": mats, "xs": xs}
    of = {"train": "pruned", "decode": case.get("of"), "encode": case.get("of")}.get(kind, kind)
    rp, ci, v, n = _matrix(case, of, gen)
    s = {"rp": rp, "ci": ci, "v": v, "n": n, "m": rp.numel() - 1}
    k = case.get("k", 1)
    if kind == "train":
        s["x"] = _uniform((k, n), dtype, gen)
        s["dy"] = _uniform((k, s["m"]), dtype, gen)
    else:
        s["x"] = _uniform((n,) if k == 1 else (n, k), dtype, gen)
    if kind == "sym":
        s["diag"] = torch.rand(n, dtype=dtype, device=DEV, generator=gen) + 1
    return s


def prepare(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    if kind == "encode":
        return {"case": dict(case), **s}
    if kind == "batch":
        mats = [P.Matrix.from_csr_device(rp, ci, v, n, layout="row", sort_window=0) if not case["sort"] else
                P.Matrix.from_csr(rp.cpu(), ci.cpu(), v.cpu(), n, layout="row", sort_window=256)
                for rp, ci, v, n in s["mats"]]
        return {"case": dict(case), "batch": P.Batch(mats), "xs": s["xs"]}
    options = {}
    if case.get("paper"):  # the paper's own format
        options = {"first_delta_column": True, "max_mult": 256}
    if case.get("in_stream"):  # the host encoder writes this form
        A = P.Matrix.from_csr(s["rp"].cpu(), s["ci"].cpu(), s["v"].cpu(), s["n"], escape_in_stream=True)
    else:
        A = P.Matrix.from_csr_device(s["rp"], s["ci"], s["v"], s["n"], **options)
    A.to_device().reserve(case.get("k", 1))
    state = {"case": dict(case), "A": A, "x": s["x"]}
    if kind == "train":
        state.update(layer=DtansLinear(A), x=s["x"].requires_grad_(), dy=s["dy"])
    if kind == "sym":
        state["diag"] = s["diag"]
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        return state["batch"].spmv(state["xs"]) if case["k"] == 1 else state["batch"].spmm(state["xs"])
    if kind == "train":
        y = state["layer"](state["x"])
        dx, = torch.autograd.grad(y, state["x"], state["dy"])
        return y, dx
    if kind == "sym":
        return state["A"].spmv_sym(state["x"], state["diag"])
    if kind == "decode":
        return state["A"].decode_csr()
    if kind == "encode":
        A = P.Matrix.from_csr_device(state["rp"], state["ci"], state["v"], state["n"])
        return A.spmv(state["x"])
    return state["A"].spmv(state["x"]) if case["k"] == 1 else state["A"].spmm(state["x"])


# ------------------------------------------------------ what a pass cannot avoid
def _nnz(case, kind):
    if kind == "band":
        return case["m"] * case["per_row"] * (1 - case["per_row"] / 1026)
    if kind == "stencil":
        return (3 * case["g"] - 2) ** 3
    if kind == "sym":
        return ((3 * case["g"] - 2) ** 3 - case["g"] ** 3) // 2
    if kind == "rmat":
        return 16.3 * 2 ** case["scale"]
    if kind == "skewed":
        return 15.0 * case["m"]
    return case["m"] * case["n"] / 2


def work(case):
    """Bytes: the compressed streams, the coding tables and row pointers, and
    the vectors, each once for each product with the matrix.  Operations: two
    for each nonzero and right-hand side."""
    kind, k, vb = case["kind"], case.get("k", 1), 8 if case["f64"] else 4
    tables = 4096 * (8 + vb)
    if kind == "batch":
        sizes = _batch_sizes(case)
        nnz = 35.0 * sum(sizes)
        return {"bytes": nnz * 2.2 + sum(sizes) * (4 + 2 * vb * k) + tables * len(sizes), "flops": 2 * nnz * k}
    of = {"train": "pruned", "decode": case.get("of"), "encode": case.get("of")}.get(kind, kind)
    nnz = _nnz(case, of)
    m = case["g"] ** 3 if "g" in case else 1 << case["scale"] if "scale" in case else case["m"]
    n = case.get("n", m)
    matrix = nnz * _BITS[of] / 8 + 4 * m + tables
    csr = nnz * (4 + vb) + 4 * m
    if kind == "train":
        return {"bytes": 2 * (matrix + (m + n) * k * vb), "flops": 4 * nnz * k}
    if kind == "sym":
        return {"bytes": matrix + 3 * m * vb, "flops": 4 * nnz + 2 * m}
    if kind == "decode":
        return {"bytes": matrix + csr, "flops": 0}
    if kind == "encode":
        return {"bytes": csr + 2 * matrix + (m + n) * vb, "flops": 2 * nnz}
    return {"bytes": matrix + (m + n) * k * vb, "flops": 2 * nnz * k}


# ------------------------------------------------------------- exact results
def _product(rp, ci, v, x, rows_out, transposed=False):
    """A x (or A^T x) in 64 bits: x of shape [n] or [n, k], a column at a time."""
    row = torch.repeat_interleave(torch.arange(rp.numel() - 1, device=DEV), torch.diff(rp.long()))
    src, dst = (row, ci.long()) if transposed else (ci.long(), row)
    w = v.double()

    def one(c):
        return torch.zeros(rows_out, dtype=torch.float64, device=DEV).index_add_(0, dst, w * c[src])

    x = x.double()
    return one(x) if x.dim() == 1 else torch.stack([one(x[:, j].contiguous()) for j in range(x.size(1))], 1)


def exact(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    if kind == "batch":
        return [_product(rp, ci, v, x, n) for (rp, ci, v, n), x in zip(s["mats"], s["xs"])]
    rp, ci, v, x = s["rp"], s["ci"], s["v"], s["x"]
    if kind == "decode":
        return rp, ci, v.double()
    if kind == "train":
        return (_product(rp, ci, v, x.t(), s["m"]).t(), _product(rp, ci, v, s["dy"].t(), s["n"], True).t())
    y = _product(rp, ci, v, x, s["m"])
    if kind == "sym":
        y = y + _product(rp, ci, v, x, s["n"], True) + s["diag"].double() * x.double()
    return y
