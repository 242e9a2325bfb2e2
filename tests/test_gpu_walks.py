"""Which walk a matrix gets, at the edges of each rule, and the walks that the other tests' matrices no longer reach:
blocks of right-hand sides over columns too far apart for 16 bits, A' and then A'^T, batches whose matrices differ."""

import numpy as np
import pytest

from gen import CsrInput
from tests.gpu_util import check_forward, params, say, to_dev
from tests.test_gpu_nonfinite import heavy_band
from tests.test_gpu_window import CASES, DT, band, symmetrised, wide

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import adjoint as OA  # noqa: E402
from oracle import precision as OP  # noqa: E402
from oracle import spmv as OS  # noqa: E402
from paper_2203_05096_amd import _capi as C  # noqa: E402
from paper_2203_05096_amd.matrix import CsrkBatch, CsrkMatrix  # noqa: E402

LANES = 2


def build(A, srs, store="f64", waves=2):
    A.vals = OP.stored_values(A.vals, store)
    return CsrkMatrix.from_csr(A.row_ptr, A.col_idx, A.vals, store=store,
                               params=params(srs, 3, lanes=LANES, waves=waves, reorder="none"))


def union_lengths(A):
    """Entries per row of A + A^T."""
    import scipy.sparse as sp
    P = sp.csr_matrix((np.ones(A.nnz), A.col_idx, A.row_ptr), shape=(A.n, A.n))
    return np.diff((P + P.T).tocsr().indptr)


def cut(sr, length):
    """The launch's windows: super-rows of at most 64 rows and 504 entries, others cut into about equal rows within
    both, a row of more than 256 entries alone."""
    out = [0]
    for r0, r1 in zip(sr[:-1], sr[1:]):
        if r1 - r0 <= 64 and length[r0:r1].sum() <= 504:
            out.append(r1)
            continue
        pieces = -(-(r1 - r0) // 64)
        rows, total, alone = -(-(r1 - r0) // pieces), 0, False
        for i in range(r0, r1):
            if i > out[-1] and (alone or length[i] > 256 or i - out[-1] == rows or total + length[i] > 504):
                out.append(i)
                total = 0
            total += length[i]
            alone = length[i] > 256
        out.append(r1)
    return np.array(out)


def due(A, M):
    """The walk that the rules give the matrix (rows in their own order, columns within 16 bits)."""
    sr = M.structure()["sr_ptr"].astype(np.int64)
    own, both = np.diff(A.row_ptr), union_lengths(A)
    sym = both.sum() == own.sum()
    sums = (lambda ptr, length: np.add.reduceat(np.append(length, 0), ptr[:-1]) * (np.diff(ptr) > 0))
    fits = (lambda ptr: np.diff(ptr).max() <= 64 and sums(ptr, both).max() <= 504)
    most = 1.4 if A.nnz <= 1 << 20 else 1.2
    win = cut(sr, both if fits(sr) or both.sum() <= most * own.sum() else own)
    longest = max(own.max(), np.bincount(A.col_idx, minlength=A.n).max())
    lanes = 1
    while lanes < 16 and np.diff(win).max() * lanes * 2 <= 64:
        lanes *= 2
    window = sums(win, own).max() <= 504 and longest <= 32 * lanes
    union = fits(win)
    one = sym or (union and (window or longest <= 16 * LANES))
    return {"windows": len(win) - 1, "product_window": int(window), "adjoint_window": int(window and (sym or union)),
            "lanes": lanes if window else 0, "adjoint_passes": 1 if one else 2}


@pytest.mark.parametrize("name", list(CASES) + ["band"])
def test_walk_of_edge_matrices(name):
    """Every field against the rules written out, for the edge matrices and bands with more and more dropped."""
    seen = []
    makes = [CASES[name]] if name in CASES else \
        [(lambda d=d: band(1203, d), srs) for d in (0.02, 0.1, 0.3, 0.5, 0.9) for srs in (40, 50, 200)]
    for make, srs in makes:
        for A in (make(), symmetrised(make())):
            M = build(A, srs)
            w = C.csrk_get_walk(M.handle)
            say("walk", name, A.name, w)
            want = due(A, M)
            assert {k: w[k] for k in want} == want
            seen.append((w["product_window"], w["adjoint_passes"]))
            M.close()
    assert name not in ("beyond", "heavy") or (0, 2) in seen
    assert name not in ("one_row", "lanes16") or seen[0][0] == 1


@pytest.mark.parametrize("n,drop", [(140000, 0.3), (190000, 0.3), (190000, 0.1), (140000, 0.6)])
def test_walk_by_extras_and_entries(n, drop):
    """Super-rows are cut for the union up to 1.4 times the entries in small matrices, 1.2 times in others; with 60%
    dropped, the union fits the super-rows all the same."""
    cols = np.arange(n)[:, None] + np.arange(-4, 5)
    keep = (cols >= 0) & (cols < n) & ((np.random.default_rng(9).random(cols.shape) >= drop) | (cols == np.arange(n)[:, None]))
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    A = CsrInput("band", n, rp, cols[keep].astype(np.int32), np.ones(keep.sum()), {})
    M = build(A, 64)
    w, want = C.csrk_get_walk(M.handle), due(A, M)
    assert {k: w[k] for k in want} == want
    assert want["adjoint_passes"] == (2 if (n, drop) == (190000, 0.3) else 1)
    M.close()


def test_walk_windows():
    """504 entries stay one window, more are cut; a handle that is not uploaded has no walk."""
    full = symmetrised(band(640, 0.0))
    for rows, windows in ((64, 20), (56, 12)):
        # bands of nine: 64 rows hold 576 entries (cut in two), 56 rows 504 (one window)
        M = build(full, rows)
        sr = M.structure()["sr_ptr"]
        assert np.array_equal(sr, np.minimum(np.arange(len(sr)) * rows, 640))
        assert C.csrk_get_walk(M.handle)["windows"] == windows
        M.close()
    h = C.csrk_build_host(full.row_ptr, full.col_idx, full.vals, params(64, 3))
    with pytest.raises(C.CsrkError) as e:
        C.csrk_get_walk(h)
    C.csrk_destroy(h)
    assert e.value.name == "CSRK_ERR_UNSUPPORTED"


def span(A, srs):
    """The widest super-row: how far its last column lies from its first."""
    sr = np.repeat(np.arange(A.n) // srs, np.diff(A.row_ptr))
    lo, hi = np.full(A.n // srs + 1, A.n), np.zeros(A.n // srs + 1, dtype=np.int64)
    np.minimum.at(lo, sr, A.col_idx)
    np.maximum.at(hi, sr, A.col_idx)
    return int((hi - lo).max())


@pytest.mark.parametrize("sym", [False, True])
def test_walk_column_span(sym):
    """Columns of a window within 65536 of each other are kept in 16 bits: those of A' for the product, those of
    A' + A'^T for the adjoint."""
    seen = set()
    for gap in (65500, 65519, 65520, 65521, 65535, 65536):
        A = wide(70001, 16, gap)
        U = symmetrised(A)
        A = U if sym else A
        M = build(A, 16)
        w = C.csrk_get_walk(M.handle)
        assert w["windows"] == (A.n + 15) // 16
        due = span(A, 16) <= 65535, span(U, 16) <= 65535
        assert (w["product_window"], w["adjoint_window"], w["adjoint_passes"]) == (*due, 1), gap
        seen.add((due, span(A, 16), span(U, 16)))
        M.close()
    assert {d for d, _, _ in seen} >= ({(True, True), (False, False)} | (set() if sym else {(True, False)}))
    assert sym or {a for _, a, _ in seen} >= {65535, 65536}


def close(out, ref, scale, beta, what):
    assert np.all(np.abs(out.double().cpu().numpy() - ref) <= beta * scale), what


def check(Ms, As, nrhs, caller):
    """Products and both gradients, alone and in one batch, within the bounds of their sums in FP64 or FP32."""
    store = Ms[0].store
    rng = np.random.default_rng(nrhs)
    shape = (lambda A: (A.n,) if nrhs == 1 else (A.n, nrhs))
    xs, gs = ([rng.uniform(-1, 1, shape(A)).astype(np.float32).astype(np.float64) for A in As] for _ in range(2))
    xd, gd = [to_dev(x, DT[store]) for x in xs], [to_dev(g, DT[store]) for g in gs]
    vals = [M.values() if caller else None for M in Ms]
    B = CsrkBatch(Ms)
    many = vals if caller else None
    yb, (bx, bv) = B.spmv(xd, vals=many), B.adjoint(xd, gd, vals=many)
    for i, (M, A) in enumerate(zip(Ms, As)):
        y, (gx, gv) = M.spmv(xd[i], vals=vals[i]), M.adjoint(xd[i], gd[i], vals=vals[i])
        torch.cuda.synchronize()
        c = np.maximum(np.bincount(A.col_idx, minlength=A.n), 1)
        c = c if nrhs == 1 else c[:, None]
        f64 = store == "f64"
        for o in (y, yb[i]):
            check_forward(o.double().cpu().numpy(), A, xs[i], np.arange(A.n), store, False, label=A.name)
        for o in (gx, bx[i]):
            close(o, OA.grad_x(A.row_ptr, A.col_idx, A.vals, gs[i]),
                  OA.grad_x(A.row_ptr, A.col_idx, np.abs(A.vals), np.abs(gs[i])),
                  1e-12 if f64 else OP.gamma(c, 2.0 ** -24), (A.name, "grad_x"))
        for o in (gv, bv[i]):
            close(o, OA.grad_vals(A.row_ptr, A.col_idx, xs[i], gs[i]),
                  OA.grad_vals(A.row_ptr, A.col_idx, np.abs(xs[i]), np.abs(gs[i])),
                  1e-12 if f64 else OP.gamma(nrhs, 2.0 ** -24), (A.name, "grad_vals"))
    B.close()


@pytest.mark.parametrize("caller", [False, True])
@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("nrhs", [1, 2, 5, 8])
@pytest.mark.parametrize("name", ["wide", "wide sym", "two passes"])
def test_general_walk(name, nrhs, store, caller):
    say("general walk", name, nrhs, store, caller)
    if name == "two passes":
        A = heavy_band()
        A.vals = np.random.default_rng(2).uniform(-1, 1, A.nnz)
        M = build(A, 30, store)
    else:
        A = wide(70001, 16, 65536)
        A = symmetrised(A) if name == "wide sym" else A
        M = build(A, 16, store)
    w = C.csrk_get_walk(M.handle)
    assert w["product_window"] == 0 and w["adjoint_passes"] == (2 if name == "two passes" else 1)
    check([M, M], [A, A], nrhs, caller)
    M.close()


@pytest.mark.parametrize("caller", [False, True])
@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("nrhs", [1, 3, 8])
@pytest.mark.parametrize("name", ["extras", "extras of long rows", "cut"])
def test_union_windows(name, nrhs, store, caller):
    """The window walk over unions: patterns without a mirror, whose rows have as many extras as entries (around one
    and several batches of them), and super-rows cut into windows for their union."""
    say("union windows", name, nrhs, store, caller)
    if name == "cut":
        A, srs = band(1203, 0.1), 200
    else:
        lengths, srs = ([1, 2, 3, 4, 5, 9, 10, 11, 13] * 50, 16) if name == "extras" else ([60, 17, 33, 64, 40, 1] * 50, 3)
        rows = [np.arange(i, min(i + m, len(lengths))) for i, m in enumerate(lengths)]  # an upper triangle
        rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
        A = CsrInput(name, len(rows), rp, np.concatenate(rows).astype(np.int32), np.zeros(rp[-1]), {})
        A.vals = np.random.default_rng(6).uniform(-1, 1, A.nnz)
    M = build(A, srs, store)
    w = C.csrk_get_walk(M.handle)
    assert w["adjoint_window"] == 1 and M.info["adjoint_union"] == (name != "cut")
    check([M, M], [A, A], nrhs, caller)
    M.close()


@pytest.mark.parametrize("caller", [False, True])
@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("nrhs", [1, 4, 5])
@pytest.mark.parametrize("mix", ["lanes", "patterns", "lanes and patterns"])
def test_batch_of_different_windows(mix, nrhs, store, caller):
    """One launch over matrices of different lanes per row, and over symmetric and nonsymmetric patterns."""
    say("batch mix", mix, nrhs, store, caller)
    if mix == "lanes":
        As, srs = [symmetrised(band(333, 0.1)) for _ in range(3)], (40, 17, 5)
    elif mix == "patterns":
        As, srs = [symmetrised(band(333, 0.1)), band(777, 0.3), symmetrised(band(64, 0.2))], (24, 24, 24)
    else:
        As, srs = [band(333, 0.1), symmetrised(band(777, 0.3)), band(65, 0.2), CASES["tiny"][0]()], (4, 9, 30, 64)
    Ms = [build(A, s, store) for A, s in zip(As, srs)]
    ws = [C.csrk_get_walk(M.handle) for M in Ms]
    assert all(w["product_window"] and w["adjoint_window"] for w in ws)
    assert (len({w["lanes"] for w in ws}) > 1) == ("lanes" in mix)
    check(Ms, As, nrhs, caller)
    for M in Ms:
        M.close()


def repeated(n, entries):
    """A symmetric band of `entries` (odd) a row: -1 off the diagonal, a dominant diagonal."""
    h = entries // 2
    cols = np.arange(n)[:, None] + np.arange(-h, h + 1)
    ok = (cols >= 0) & (cols < n)
    rp = np.concatenate([[0], np.cumsum(ok.sum(1))]).astype(np.int32)
    ci = cols[ok].astype(np.int32)
    vals = np.where(ci == np.repeat(np.arange(n), np.diff(rp)), entries + 1.0, -1.0)
    return CsrInput("band", n, rp, ci, vals, {})


@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("n,entries,launches", [(100000, 31, 2), (105000, 31, 3), (393216, 5, 2), (393217, 5, 3),
                                                (393000, 9, 3)])
def test_cg_launches_by_entries_and_rows(n, entries, launches, store):
    """Two launches an iteration up to 3 * 2^20 entries and 3 * 2^17 rows: many entries in few rows take three.  The
    solve is checked by the residual of the stored matrix (exact values): the recurrence drifts from it by rounding
    alone in FP64 (2x the tolerance), by the FP32 products otherwise (100x)."""
    say("cg launches", n, entries, store)
    A = repeated(n, entries)
    M = CsrkMatrix.from_csr(A.row_ptr, A.col_idx, A.vals, store=store)
    assert C.csrk_get_walk(M.handle)["cg_launches"] == launches
    perm = M.structure()["perm"]
    b, rtol = np.random.default_rng(4).uniform(-1, 1, n), 1e-6
    x, it, rel = M.cg(to_dev(b[perm], torch.float64), rtol=rtol, max_iter=500, check_every=5)
    assert 0 < it < 500 and rel <= rtol
    xin = np.empty(n)
    xin[perm] = x.cpu().numpy()
    res = np.linalg.norm(b - OS.spmv(A.row_ptr, A.col_idx, A.vals, xin)) / np.linalg.norm(b)
    assert res <= (2 if store == "f64" else 100) * rtol, res
    M.close()


@pytest.mark.parametrize("sym", [True, False])
@pytest.mark.parametrize("store,nrhs,n", [("f32", 130, 110000), ("f64", 8, 600000), ("bf16", 16, 800000),
                                          ("f32", 5, 1600000)])
def test_block_launches_past_the_caches(store, nrhs, n, sym):
    """Blocks whose launches move more than 96 MB read the handle's values past the caches: both directions, exact and
    overlapping slices, one and several chunks of columns, symmetric patterns and unions."""
    say("large block", store, nrhs, n, sym)
    rng = np.random.default_rng(nrhs)
    cols = np.arange(n)[:, None] + np.arange(-2, 3)
    keep = (cols >= 0) & (cols < n) & (sym | (rng.random(cols.shape) >= 0.1) | (cols == np.arange(n)[:, None]))
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    A = CsrInput("large", n, rp, cols[keep].astype(np.int32), np.round(rng.uniform(-1, 1, keep.sum()) * 64) / 64, {})
    vb, xb = {"f64": (8, 8), "f32": (4, 4), "bf16": (2, 4)}[store]
    assert A.nnz * (vb + 2) + 2 * n * nrhs * xb > 96 << 20
    M = CsrkMatrix.from_csr(A.row_ptr, A.col_idx, A.vals, store=store, nrhs=nrhs, params=params(32, 4, reorder="none"))
    w = C.csrk_get_walk(M.handle)
    assert w["product_window"] and w["adjoint_window"]
    x, g = (rng.uniform(-1, 1, (n, nrhs)).astype(np.float32).astype(np.float64) for _ in range(2))
    xd, gd = to_dev(x, DT[store]), to_dev(g, DT[store])
    y, (gx, gv) = M.spmv(xd), M.adjoint(xd, gd)
    _, only = M.adjoint(xd, gd, grad_x=False)
    torch.cuda.synchronize()
    check_forward(y.double().cpu().numpy(), A, x, np.arange(n), store, False, label="large block")
    f64 = store == "f64"
    c = np.maximum(np.bincount(A.col_idx, minlength=n), 1)[:, None]
    close(gx, OA.grad_x(A.row_ptr, A.col_idx, A.vals, g), OA.grad_x(A.row_ptr, A.col_idx, np.abs(A.vals), np.abs(g)),
          1e-12 if f64 else OP.gamma(c, 2.0 ** -24), "grad_x")
    ref, scale = OA.grad_vals(A.row_ptr, A.col_idx, x, g), OA.grad_vals(A.row_ptr, A.col_idx, np.abs(x), np.abs(g))
    for o in (gv, only):
        close(o, ref, scale, 1e-12 if f64 else OP.gamma(nrhs, 2.0 ** -24), "grad_vals")
    M.close()


@pytest.mark.parametrize("objective", ["forward", "step"])
def test_sweep_times_equal_launches_once(objective):
    """Trials that differ in lanes per row only, where the launch does not read them, are one launch and one timing:
    window walks and blocks of right-hand sides.  The general walk's lanes are each timed."""
    from paper_2203_05096_amd import autotune as T
    general = wide(70001, 16, 65536)
    for A, nrhs, same in ((band(3000, 0.1), 1, True), (general, 4, True), (general, 1, False)):
        say("sweep lanes", A.name, nrhs, objective)
        res = T.sweep(A, "f64", srs_list=(16, 32), ssrs_list=(2,), lanes_list=(1, 2, 4), nrhs=nrhs, reps=20, threads=2,
                      reorder="none", objective=objective)
        assert len(res.trials) == 6
        for srs in (16, 32):
            times = {t.us for t in res.trials if t.srs == srs}
            assert len(times) == 1 if same else len(times) > 1
        assert not same or res.best.lanes == 1
