"""The window walk at the edges of its rule: full and overfull windows, column spans around 16 bits, rows around a
batch of gathers, empty rows and super-rows, windows that start and end off a load boundary, super-rows cut into
windows; against the oracle."""

import numpy as np
import pytest

from gen import CsrInput
from tests.gpu_util import check_forward, params, say, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import adjoint as OA  # noqa: E402
from oracle import precision as OP  # noqa: E402
from oracle import spmv as OS  # noqa: E402
from paper_2203_05096_amd.matrix import CsrkBatch, CsrkMatrix  # noqa: E402

DT = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.float32}


def matrix(lengths, n=None, seed=0, span=None):
    """Rows of the given lengths with random columns (the first `span` columns of a row's neighbourhood)."""
    rng = np.random.default_rng(seed)
    n = len(lengths) if n is None else n
    cols = []
    for i, m in enumerate(lengths):
        w = n if span is None else span
        lo = min(max(0, i - w // 2), n - w)
        cols.append(np.sort(rng.choice(w, m, replace=False)) + lo)
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = np.concatenate(cols).astype(np.int32) if len(cols) else np.zeros(0, np.int32)
    return CsrInput("w", n, rp, ci, rng.uniform(-1, 1, len(ci)), {})


def wide(n, srs, gap):
    """A band of three, and in the first row of each super-row an entry `gap` columns away from its first column."""
    rows = [sorted({max(0, i - 1), i, min(n - 1, i + 1)}) for i in range(n)]
    for i in range(0, n, srs):
        far = rows[i][0] + gap
        if far < n:
            rows[i] = sorted(set(rows[i]) | {far})
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    return CsrInput("wide", n, rp, ci, np.random.default_rng(3).uniform(-1, 1, len(ci)), {})


CASES = {
    # 64 rows; 7 and 8 entries: one batch; 504 entries fill the window, 505 do not fit
    "full": (lambda: matrix([8] * 63 + [0] + [7] * 64 + [8] * 62 + [4, 4]), 64),
    "overfull": (lambda: matrix([8] * 62 + [9, 0] + [7] * 64), 64),
    # rows around one and two batches of one lane, up to the four batches of the rule, and beyond it
    "batches": (lambda: matrix([9, 15, 16, 17, 31, 32, 8, 0] * 13 + [5]), 33),
    "beyond": (lambda: matrix([3] * 40 + [33] + [2] * 60), 40),
    # two to sixteen lanes per row, with short last super-rows
    "lanes2": (lambda: matrix([15, 17, 13, 0] * 21 + [16]), 32),
    "lanes4": (lambda: matrix([27, 31, 33, 25, 32] * 20 + [64]), 15),
    "lanes8": (lambda: matrix([64, 63, 65, 50, 56, 1] * 20 + [9]), 7),
    "lanes16": (lambda: matrix([128, 127, 129, 100] * 40 + [3]), 3),
    "one_row": (lambda: matrix([200, 0, 1, 7, 33, 180] * 40), 1),
    # super-rows cut into windows: more rows or entries than one holds, heavy and long rows alone
    "rows96": (lambda: matrix([3, 4, 5, 2] * 130), 96),
    "cut": (lambda: matrix([14, 16, 9, 31] * 50), 50),
    "heavy": (lambda: matrix(([2] * 30 + [300, 129, 128, 505] + [3] * 51) * 20 + [1500, 1024, 1025] + [7] * 5), 64),
    "empty": (lambda: matrix([0] * 64 + [3] * 64 + [0] * 70), 64),
    "tiny": (lambda: matrix([1, 0, 2]), 64),
}


def check_adjoint(M, A, x, g, B, vals):
    """Both gradients (alone and batched): grad_x within 1e-12 (FP64) or gamma_c(2^-24) of the oracle's, c a column's
    entries; grad_vals, one rounded product per entry, equal to it."""
    store = M.store
    xd, gd = to_dev(x, DT[store]), to_dev(g, DT[store])
    gx, gv = M.adjoint(xd, gd, vals=vals)
    bx, bv = B.adjoint([xd, xd], [gd, gd], vals=None if vals is None else [vals, vals])
    torch.cuda.synchronize()
    ref = OA.grad_x(A.row_ptr, A.col_idx, A.vals, g)
    scale = OA.grad_x(A.row_ptr, A.col_idx, np.abs(A.vals), np.abs(g))
    c = np.maximum(np.bincount(A.col_idx, minlength=A.n), 1)
    beta = 1e-12 if store == "f64" else OP.gamma(c, 2.0 ** -24)
    for out in (gx, bx[0]):
        assert np.all(np.abs(out.double().cpu().numpy() - ref) <= beta * scale)
    refv = OA.grad_vals(A.row_ptr, A.col_idx, x, g)
    refv = refv if store == "f64" else refv.astype(np.float32).astype(np.float64)
    assert np.array_equal(gv.double().cpu().numpy(), refv)
    assert torch.equal(bx[0], bx[1]) and torch.equal(bv[0], gv) and torch.equal(bv[1], gv)


def symmetrised(A):
    import scipy.sparse as sp
    P = sp.csr_matrix((np.ones(A.nnz), A.col_idx, A.row_ptr), shape=(A.n, A.n))
    P = (P + P.T).tocsr()
    P.sort_indices()
    return CsrInput("sym", A.n, P.indptr.astype(np.int32), P.indices.astype(np.int32),
                    np.random.default_rng(7).uniform(-1, 1, P.nnz), {})


def check(A, srs, store, waves):
    A.vals = OP.stored_values(A.vals, store)
    M = CsrkMatrix.from_csr(A.row_ptr, A.col_idx, A.vals, store=store,
                            params=params(srs, 3, lanes=2, waves=waves, reorder="none"))
    x, g = np.random.default_rng(1).uniform(-1, 1, (2, A.n)).astype(np.float32).astype(np.float64)
    xd = to_dev(x, DT[store])
    y = M.spmv(xd)
    y2 = M.spmv(xd, vals=M.values())
    B = CsrkBatch([M, M])
    yb = B.spmv([xd, xd])
    torch.cuda.synchronize()
    # the general walk sums long rows in another order alone than batched: each against the oracle
    for out in (y, yb[0]):
        check_forward(out.double().cpu().numpy(), A, x, np.arange(A.n), store, False, label="window")
    assert torch.equal(y, y2) and torch.equal(yb[0], yb[1])
    for vals in (None, M.values()):
        check_adjoint(M, A, x, g, B, vals)
    B.close()
    M.close()


@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("name", list(CASES))
def test_window_edges(name, store):
    make, srs = CASES[name]
    for A in (make(), symmetrised(make())):
        say("window", name, store, A.name)
        check(A, srs, store, waves=2)


@pytest.mark.parametrize("gap", [65535, 65536])
@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
def test_window_column_span(gap, store):
    """Column offsets up to 65535 are 16-bit; one more and the general walk takes the matrix."""
    say("window span", gap, store)
    check(wide(70001, 16, gap), 16, store, waves=4)


def band(n, drop, seed=5):
    """A band of nine with entries dropped: nonsymmetric, short extras per row."""
    rng = np.random.default_rng(seed)
    rows = [[j for j in range(max(0, i - 4), min(n, i + 5)) if j == i or rng.random() >= drop] for i in range(n)]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    return CsrInput("band", n, rp, ci, rng.uniform(-1, 1, len(ci)), {})


@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("srs,drop", [(40, 0.1), (48, 0.5), (17, 0.3), (8, 0.2), (3, 0.1)])
def test_window_union(srs, drop, store):
    """Nonsymmetric patterns whose union fits the window, every number of lanes per row."""
    say("window union", srs, drop, store)
    check(band(1203, drop), srs, store, waves=3)


def block(a, store, shift):
    """The block on the GPU, `shift` elements into its allocation."""
    raw = torch.empty(a.size + shift, dtype=DT[store], device="cuda")
    raw[shift:] = to_dev(a, DT[store]).reshape(-1)
    return raw[shift:].view(a.shape)


@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("nrhs,shift", [(2, 0), (3, 1), (4, 1), (5, 0), (8, 0), (13, 1), (33, 0), (65, 1), (130, 0)])
@pytest.mark.parametrize("name", ["full", "batches", "lanes2", "lanes4", "lanes16", "rows96", "tiny", "band"])
def test_window_blocks(name, nrhs, shift, store):
    """Blocks of right-hand sides: slices that end off a slice boundary, blocks off 16 bytes, several chunks of columns.
    Forward and grad_x within the bounds of one column; grad_vals, a sum over the columns, within gamma_nrhs."""
    make, srs = CASES[name] if name != "band" else (lambda: band(407, 0.2), 24)
    for A in (make(), symmetrised(make())):
        say("window blocks", name, nrhs, shift, store, A.name)
        A.vals = OP.stored_values(A.vals, store)
        M = CsrkMatrix.from_csr(A.row_ptr, A.col_idx, A.vals, store=store,
                                params=params(srs, 3, lanes=2, waves=2, reorder="none"))
        X, G = np.random.default_rng(nrhs).uniform(-1, 1, (2, A.n, nrhs)).astype(np.float32).astype(np.float64)
        x, g = block(X, store, shift), block(G, store, shift)
        B = CsrkBatch([M, M])
        for vals in (None, M.values()):
            two = None if vals is None else [vals, vals]
            gx, gv = M.adjoint(x, g, vals=vals)
            only = M.adjoint(x, g, vals=vals, grad_x=False)[1]
            ys = [M.spmv(x, vals=vals)] + B.spmv([x, x], vals=two)
            bx, bv = B.adjoint([x, x], [g, g], vals=two)
            torch.cuda.synchronize()
            for y in ys:
                check_forward(y.double().cpu().numpy(), A, X, np.arange(A.n), store, False, label="window block")
            ref = OA.grad_x(A.row_ptr, A.col_idx, A.vals, G)
            scale = OA.grad_x(A.row_ptr, A.col_idx, np.abs(A.vals), np.abs(G))
            c = np.maximum(np.bincount(A.col_idx, minlength=A.n), 1)[:, None]
            beta = 1e-12 if store == "f64" else OP.gamma(c, 2.0 ** -24)
            for out in [gx] + bx:
                assert np.all(np.abs(out.double().cpu().numpy() - ref) <= beta * scale)
            ref = OA.grad_vals(A.row_ptr, A.col_idx, X, G)
            scale = OA.grad_vals(A.row_ptr, A.col_idx, np.abs(X), np.abs(G))
            beta = 1e-12 if store == "f64" else OP.gamma(nrhs, 2.0 ** -24)
            for out in [gv, only] + bv:
                assert np.all(np.abs(out.double().cpu().numpy() - ref) <= beta * scale)
        B.close()
        M.close()


@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("side,band_rows", [(16, 0), (0, 500000)])
def test_cg_launch_rules(side, band_rows, store):
    """CG with two launches an iteration (a small grid) and with three (more rows than that rule takes), checked by the
    residual of the stored matrix: the recurrence drifts from it by the FP32 rounding of the products at most (100x the
    tolerance), in FP64 storage by rounding alone (2x).  Twice on one handle, which keeps its work memory: equal bits."""
    if side:
        from gen import laplacian
        A = laplacian((side, side + 1, side + 3), "3d7", 6.0)
    else:
        n = band_rows
        rp = np.concatenate([[0], np.cumsum(np.r_[2, np.full(n - 2, 3), 2])]).astype(np.int32)
        ci = np.concatenate([[0, 1], (np.arange(1, n - 1)[:, None] + [-1, 0, 1]).ravel(), [n - 2, n - 1]]).astype(np.int32)
        A = CsrInput("tri", n, rp, ci, np.where(ci == np.repeat(np.arange(n), np.diff(rp)), 4.0, -1.0), {})
    say("cg launches", A.n, store)
    M = CsrkMatrix.from_csr(A.row_ptr, A.col_idx, A.vals, store=store)
    perm = M.structure()["perm"]
    b = np.random.default_rng(4).uniform(-1, 1, A.n)
    bd = to_dev(b[perm], torch.float64)
    rtol = 1e-6
    x, it, rel = M.cg(bd, rtol=rtol, max_iter=500, check_every=7)
    x2, it2, rel2 = M.cg(bd, rtol=rtol, max_iter=500, check_every=7)
    torch.cuda.synchronize()
    assert it == it2 and rel == rel2 and torch.equal(x, x2)
    assert 0 < it < 500 and it % 7 == 0 and rel <= rtol
    xin = np.empty(A.n)
    xin[perm] = x.cpu().numpy()
    res = np.linalg.norm(b - OS.spmv(A.row_ptr, A.col_idx, A.vals, xin)) / np.linalg.norm(b)
    assert res <= (2 if store == "f64" else 100) * rtol, res
    x, it, rel = M.cg(bd, x0=x, rtol=rtol, max_iter=500, check_every=1)  # from the solution: at most a few iterations
    assert it <= 7
    M.close()


@pytest.mark.parametrize("rows", [1 << 19, (1 << 19) + 1, (1 << 20) + 4097])
@pytest.mark.parametrize("store", ["f64", "f32"])
def test_cg_large_workgroups(rows, store):
    """The passes over the vectors at the last row count of the small workgroups, the first of the large ones, and one
    that takes every large workgroup around a second time; checked as above."""
    test_cg_launch_rules(0, rows, store)
