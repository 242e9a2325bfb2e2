"""Timed cases of the CSR-k library: what a program that uses it does on the GPU.

The matrices are the ones of this repository's generators and benchmark: 2D 5-
and 9-point and 3D 7-, 19- and 27-point stencils, stencils with dropped
off-diagonals (nonsymmetric patterns) and symmetrised R-MAT graphs, from 4,096
rows up to the 2M rows of the benchmark's matrices, in the three storage
types.  A case is a plain dict:

  op     "spmv"     y = A x
         "adjoint"  grad_x = A^T g and grad_vals = g_i x_j
         "step"     one product and one adjoint, the benchmark's step
         "train"    forward and backward through CsrkSpMV with the values as a
                    parameter tensor, the autograd user's step
         "cg"       a fixed number of conjugate-gradient iterations
  kind   stencil name, or "rmat"
  dims   grid sides as text ("128x128x128"), for "rmat" the scale (n = 2^scale)
  drop   share of the off-diagonals that is left out (0: the full stencil)
  store  "f64", "f32" or "bf16"
  nrhs   right-hand sides
  count  1, or the number of matrices of a batch (sides spread from lo to hi)

Vectors and products are in the matrix's own row order, as in a solver loop:
to_permuted/from_permuted are called once, outside it.
"""

from __future__ import annotations

import itertools
import math

import numpy as np
import torch

from paper_2203_05096_amd import _capi as C
from paper_2203_05096_amd.matrix import CsrkBatch, CsrkMatrix, CsrkSpMV

_VAL = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
_VEC = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.float32}
_VBYTES = {"f64": 8, "f32": 4, "bf16": 2}
_XBYTES = {"f64": 8, "f32": 4, "bf16": 4}
_CG_ITERATIONS = 50

_BOX2 = list(itertools.product((-1, 0, 1), repeat=2))
_BOX3 = list(itertools.product((-1, 0, 1), repeat=3))
_STENCILS = {
    "2d5": [o for o in _BOX2 if sum(map(abs, o)) <= 1],
    "2d9": _BOX2,
    "3d7": [o for o in _BOX3 if sum(map(abs, o)) <= 1],
    "3d19": [o for o in _BOX3 if sum(map(abs, o)) <= 2],
    "3d27": _BOX3,
}


def _case(name, op, kind, dims, store, nrhs=1, drop=0.0, count=1, lo=0, hi=0):
    c = {"op": op, "kind": kind, "dims": dims, "store": store, "nrhs": nrhs, "drop": drop, "count": count, "lo": lo,
         "hi": hi}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest matrix of the suite: one launch, all of it in cache; a call's latency
        _case("spmv_2d5_64_f64", "spmv", "2d5", "64x64", "f64"),
        # a small problem differentiated by autograd, nonsymmetric pattern, ragged grid
        _case("train_2d9_drop_301_f32", "train", "2d9", "301x257", "f32", drop=0.1),
        # a solver's inner loop: 50 iterations on a mid-sized 3D grid
        _case("cg_3d7_64_f64", "cg", "3d7", "64x64x64", "f64"),
        # the product of the benchmark's 3D 7-point matrix, 2.1M rows
        _case("spmv_3d7_128_f64", "spmv", "3d7", "128x128x128", "f64"),
        # its adjoint (symmetric pattern) on a grid with odd sides
        _case("adjoint_3d7_odd_f64", "adjoint", "3d7", "101x97x113", "f64"),
        # the densest stencil in the smallest storage type
        _case("spmv_3d27_bf16", "spmv", "3d27", "87x90x91", "bf16"),
        # the densest stencil's adjoint
        _case("adjoint_3d27_f32", "adjoint", "3d27", "75x80x77", "f32"),
        # adjoint of a nonsymmetric pattern
        _case("adjoint_2d9_drop_f32", "adjoint", "2d9", "1201x999", "f32", drop=0.1),
        # power-law rows (web and social graphs), both directions
        _case("step_rmat_18_f64", "step", "rmat", "18", "f64"),
        # a block of right-hand sides, both directions
        _case("step_3d19_rhs8_f32", "step", "3d19", "61x64x67", "f32", nrhs=8),
        # an odd number of right-hand sides, FP64
        _case("step_2d5_rhs5_f64", "step", "2d5", "707x601", "f64", nrhs=5),
        # the benchmark's headline step at a smaller count: many 7-point matrices of uneven size, 8 right-hand sides
        _case("batch_3d7_rhs8_f32", "step", "3d7", "", "f32", nrhs=8, count=16, lo=16, hi=72),
    ]


def draw(rng):
    """One more case: any op, pattern, storage type and block width, row counts spread over their logarithm."""
    what = rng.choice(["spmv", "adjoint", "step", "train", "cg", "batch"])
    store = rng.choice(["f64", "f32", "bf16"])
    nrhs = rng.choice([1, 1, 1, 2, 3, 4, 5, 8, 12])
    if what == "batch":
        lo = rng.randint(8, 24)
        return _case("", rng.choice(["spmv", "adjoint", "step"]), "3d7", "", store, nrhs=nrhs,
                     drop=rng.choice([0.0, 0.0, 0.1]), count=rng.randint(3, 20), lo=lo, hi=lo + rng.randint(4, 32))
    if what == "cg":
        s = [int(round(2 ** rng.uniform(3.5, 6.2))) for _ in range(3)]
        return _case("", "cg", "3d7", "x".join(map(str, s)), "f64")
    if what == "train":
        store = rng.choice(["f64", "f32"])  # autograd takes the value gradients of these two
        nrhs = 1
    if rng.random() < 0.15:
        return _case("", what, "rmat", str(rng.randint(12, 17)), store, nrhs=1 if nrhs > 5 else nrhs)
    kind = rng.choice(list(_STENCILS))
    dense = len(_STENCILS[kind])
    top = min(8e6 / dense, 3e8 / (nrhs * _XBYTES[store] * 5 + dense * 20))
    rows = math.exp(rng.uniform(math.log(4096), math.log(top)))
    d = 2 if kind.startswith("2d") else 3
    side = rows ** (1.0 / d)
    f = [rng.uniform(0.8, 1.25) for _ in range(d - 1)]
    sides = [max(4, int(side * v)) for v in f] + [max(4, int(side / math.prod(f)))]
    return _case("", what, kind, "x".join(map(str, sides)), store, nrhs=nrhs, drop=rng.choice([0.0, 0.0, 0.1, 0.3]))


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(g, shape, dtype, lo=-1.0, hi=1.0):
    return torch.empty(shape, dtype=torch.float64, device="cuda").uniform_(lo, hi, generator=g).to(dtype)


def _grids(case):
    """Grid sides of each matrix of the case."""
    if case["count"] == 1:
        return [tuple(int(v) for v in case["dims"].split("x"))]
    n, lo, hi = case["count"], case["lo"], case["hi"]
    # sides spread evenly from lo to hi, in an order that mixes large and small
    return [(lo + round((hi - lo) * (b * 7 % n if n % 7 else b) / max(1, n - 1)),) * 3 for b in range(n)]


def _stencil(dims, kind):
    """(rows, cols) of a stencil on a grid, x fastest, columns increasing within a row."""
    strides = [1]
    for d in dims[:-1]:
        strides.append(strides[-1] * d)
    offs = sorted((sum(o * s for o, s in zip(off, strides)), off) for off in _STENCILS[kind])
    idx = torch.arange(math.prod(dims), device="cuda")
    coord = [(idx // s) % d for s, d in zip(strides, dims)]
    ok = torch.stack([torch.stack([(c + o >= 0) & (c + o < d) for c, o, d in zip(coord, off, dims)]).all(0)
                      for _, off in offs], 1)
    cols = idx[:, None] + torch.tensor([v for v, _ in offs], device="cuda")[None, :]
    return idx[:, None].expand_as(ok)[ok], cols[ok]


def _rmat(scale, g, edge_factor=4, probs=(0.57, 0.19, 0.19)):
    """(rows, cols) of a symmetrised R-MAT graph with the diagonal."""
    n = 1 << scale
    m = edge_factor * n
    r = torch.zeros(m, dtype=torch.int64, device="cuda")
    c = torch.zeros(m, dtype=torch.int64, device="cuda")
    cum = torch.tensor(np.cumsum(probs), device="cuda")
    for level in range(scale):
        q = torch.searchsorted(cum, torch.rand(m, dtype=torch.float64, device="cuda", generator=g), right=True)
        bit = 1 << (scale - 1 - level)
        r += torch.where(q >= 2, bit, 0)
        c += torch.where((q == 1) | (q == 3), bit, 0)
    d = torch.arange(n, device="cuda")
    key = torch.unique(torch.cat([r * n + c, c * n + r, d * n + d]))
    return key // n, key % n


def _matrix(case, dims, g):
    """(row_ptr, rows, cols, vals) on the GPU.  The pattern (mesh or graph) is the case's own; the values come from g and
    are exact in the storage type: off-diagonals -U[0.5, 1.5] in steps of 2^-16 (so that their sums are exact in any
    order) and a dominant diagonal; for cg and batches the Laplacian's -1 and 6, for cg with up to 0.1 on the diagonal."""
    mesh = _gen(4)
    if case["kind"] == "rmat":
        n = 1 << int(case["dims"])
        rows, cols = _rmat(int(case["dims"]), mesh)
    else:
        n = math.prod(dims)
        rows, cols = _stencil(dims, case["kind"])
    if case["drop"] > 0:
        keep = (rows == cols) | (torch.rand(rows.shape, device="cuda", generator=mesh) >= case["drop"])
        rows, cols = rows[keep], cols[keep]
    diag = rows == cols
    vals = -torch.round(_uniform(g, rows.shape, torch.float64, 0.5, 1.5) * 65536) / 65536
    if case["op"] == "cg" or case["count"] > 1:
        vals = torch.full_like(vals, -1.0)
        vals[diag] = 6.0 + (_uniform(g, (n,), torch.float64, 0.0, 0.1) if case["op"] == "cg" else 0.0)
    else:
        vals[diag] = 1.1 * torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(
            0, rows, torch.where(diag, 0.0, -vals)) + 0.1
    vals = vals.to(_VAL[case["store"]])
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return row_ptr, rows, cols, vals


def _inputs(case, seed):
    """Per matrix: (row_ptr, rows, cols, vals, x, g); x and g in the matrix's own row order."""
    gen = _gen(seed)
    grids = [None] if case["kind"] == "rmat" else _grids(case)
    out = []
    for dims in grids:
        row_ptr, rows, cols, vals = _matrix(case, dims, gen)
        n = row_ptr.numel() - 1
        shape = (n,) if case["nrhs"] == 1 else (n, case["nrhs"])
        out.append((row_ptr, rows, cols, vals, _uniform(gen, shape, _VEC[case["store"]]),
                    _uniform(gen, shape, _VEC[case["store"]])))
    return out


def _host(row_ptr, cols, vals):
    return (row_ptr.to(torch.int32).cpu().numpy(), cols.to(torch.int32).cpu().numpy(), vals.double().cpu().numpy())


def prepare(case, seed):
    mats, xs, gs = [], [], []
    for row_ptr, _, cols, vals, x, g in _inputs(case, seed):
        mats.append(CsrkMatrix.from_csr(*_host(row_ptr, cols, vals), store=case["store"], nrhs=case["nrhs"]))
        xs.append(x)
        gs.append(g)
    s = {"op": case["op"], "batch": None, "mats": mats, "xs": xs, "gs": gs}
    if case["count"] > 1:
        s["batch"] = CsrkBatch(mats)
    if case["op"] == "train":
        s["vals"] = mats[0].values().requires_grad_(True)
        xs[0].requires_grad_(True)
    return s


def run(state):
    op, M, x, g = state["op"], state["mats"][0], state["xs"][0], state["gs"][0]
    if state["batch"] is not None:
        B, xs, gs = state["batch"], state["xs"], state["gs"]
        if op == "spmv":
            return B.spmv(xs)
        if op == "adjoint":
            return B.adjoint(xs, gs)
        return B.spmv(xs), B.adjoint(xs, gs)
    if op == "spmv":
        return M.spmv(x)
    if op == "adjoint":
        return M.adjoint(x, g)
    if op == "step":
        return M.spmv(x), M.adjoint(x, g)
    if op == "train":
        y = CsrkSpMV.apply(M, state["vals"], x)
        gv, gx = torch.autograd.grad(y, (state["vals"], x), g)
        return y.detach(), gx, gv
    return M.cg(g, rtol=1e-14, max_iter=_CG_ITERATIONS)


# ------------------------------------------------------------------ what a pass cannot do without

def _sizes(case):
    """Rows and stored entries over all matrices of the case (expected, where entries are dropped or drawn)."""
    if case["kind"] == "rmat":
        n = 1 << int(case["dims"])
        return n, int(n * (1 + 8 * 0.96))
    n = nnz = 0
    for dims in _grids(case):
        n += math.prod(dims)
        full = sum(math.prod(d - abs(o) for d, o in zip(dims, off)) for off in _STENCILS[case["kind"]])
        nnz += full - int(case["drop"] * (full - math.prod(dims)))
    return n, nnz


def work(case):
    n, nnz = _sizes(case)
    k, vb, xb = case["nrhs"], _VBYTES[case["store"]], _XBYTES[case["store"]]
    fwd = nnz * (vb + 4) + n * (4 + 2 * k * xb)
    adj = nnz * (vb + 4 + xb) + n * (4 + 3 * k * xb)
    ops = {"spmv": (fwd, 2), "adjoint": (adj, 3), "step": (fwd + adj, 5), "train": (fwd + adj, 5)}
    if case["op"] == "cg":
        # a product, p.q (p and q just read and written), r -= alpha q with r.r, x += alpha p, p = r + beta p
        it = _CG_ITERATIONS
        return {"bytes": it * (fwd + n * 8 * 7), "flops": it * (2 * nnz + 10 * n)}
    b, f = ops[case["op"]]
    return {"bytes": b, "flops": f * nnz * k}


# ------------------------------------------------------------------ the same in 64 bits

def _layout(case, row_ptr, cols):
    """The row order that the library chose for this pattern (which row of the input each row is, and which input
    entry each stored entry is): where the values are put, not what they are."""
    rp, ci = row_ptr.to(torch.int32).cpu().numpy(), cols.to(torch.int32).cpu().numpy()
    h = C.csrk_build_host(rp, ci, None, C.csrk_tune_rhs(len(rp) - 1, len(ci), case["nrhs"]))
    s = C.csrk_copy_structure(h)
    C.csrk_destroy(h)
    return torch.from_numpy(s["perm"].astype(np.int64)).cuda(), torch.from_numpy(s["vmap"]).cuda()


def _sum_rows(to, terms, n):
    return torch.zeros((n,) + terms.shape[1:], dtype=torch.float64, device="cuda").index_add_(0, to, terms)


def exact(case, seed):
    ys, gxs, gvs = [], [], []
    for row_ptr, rows, cols, vals, x, g in _inputs(case, seed):
        n = x.shape[0]
        perm, vmap = _layout(case, row_ptr, cols)
        new = torch.empty_like(perm)
        new[perm] = torch.arange(n, device="cuda")
        i, j, a = new[rows[vmap]], new[cols[vmap]], vals[vmap].double()
        x, g = x.double(), g.double()
        wide = (slice(None),) + (None,) * (x.dim() - 1)
        if case["op"] == "cg":
            return _cg(lambda v: _sum_rows(i, a * v[j], n), g)
        if case["op"] != "adjoint":
            ys.append(_sum_rows(i, a[wide] * x[j], n))
        if case["op"] != "spmv":
            gxs.append(_sum_rows(j, a[wide] * g[i], n))
            gvs.append(g[i] * x[j] if x.dim() == 1 else (g[i] * x[j]).sum(1))
    if case["count"] == 1:
        ys, gxs, gvs = (v[0] if v else None for v in (ys, gxs, gvs))
    if case["op"] == "train":
        return ys, gxs, gvs
    return {"spmv": ys, "adjoint": (gxs, gvs), "step": (ys, (gxs, gvs))}[case["op"]]


def _cg(times, b):
    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rr = r @ r
    for _ in range(_CG_ITERATIONS):
        q = times(p)
        alpha = rr / (p @ q)
        x += alpha * p
        r -= alpha * q
        new = r @ r
        p = r + new / rr * p
        rr = new
    return x, _CG_ITERATIONS, float(torch.sqrt(rr) / torch.linalg.norm(b))
