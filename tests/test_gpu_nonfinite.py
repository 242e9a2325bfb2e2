"""Infinite and NaN entries in the vectors and values: they reach exactly the results whose sums hold a stored entry
times them (a stored zero times an infinity too), never through an entry that the matrix or its transpose does not
store.  Every walk of the product and the adjoint, against the oracle entry by entry."""

import numpy as np
import pytest

from gen import CsrInput
from tests.gpu_util import params, say, to_dev
from tests.test_gpu_window import DT, band, symmetrised, wide

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import adjoint as OA  # noqa: E402
from oracle import precision as OP  # noqa: E402
from oracle import spmv as OS  # noqa: E402
from paper_2203_05096_amd.matrix import CsrkBatch, CsrkMatrix  # noqa: E402

# A NaN that a union entry without a mirror is marked by, as a stored value: FP64, and FP32 or BF16 widened to FP64.
MARK = {"f64": 0x7FFF000000000000, "f32": 0x7FFFE00000000000, "bf16": 0x7FFFE00000000000}


def heavy_band():
    """A nonsymmetric band, and a row of 700 entries: its window's union fits no staging window."""
    B = band(1500, 0.2)
    rows = [B.col_idx[B.row_ptr[i]:B.row_ptr[i + 1]] for i in range(B.n)]
    rows[600] = np.union1d(rows[600], np.arange(2, 1402, 2)).astype(np.int32)
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    return CsrInput("heavy", B.n, rp, np.concatenate(rows), np.zeros(rp[-1]), {})


CASES = {
    "union": (lambda: band(407, 0.2), 24),  # super-rows that fit their window
    "cut": (lambda: band(407, 0.1), 200),  # cut into windows that do
    "wide": (lambda: wide(70001, 16, 65536), 16),  # columns too far apart for 16 bits
    "two passes": (heavy_band, 30),
    "symmetric": (lambda: symmetrised(band(407, 0.2)), 24),
    "symmetric wide": (lambda: symmetrised(wide(70001, 16, 65536)), 16),
}


def spoil(a, rng):
    """An infinity of each sign and a NaN in one row of sixteen, in one column of a block."""
    flat = a.reshape(len(a), -1)
    for v in (np.inf, -np.inf, np.nan):
        at = rng.choice(len(a), max(1, len(a) // 48), replace=False)
        flat[at, rng.integers(0, flat.shape[1], len(at))] = v


def same(out, ref, scale, beta, what):
    out = out.double().cpu().numpy()
    for name, f in (("NaN", np.isnan), ("+inf", np.isposinf), ("-inf", np.isneginf)):
        assert np.array_equal(f(out), f(ref)), f"{what}: {name} in {int(f(out).sum())} entries, {int(f(ref).sum())} due"
    fin = np.isfinite(ref)
    assert np.all(np.abs(out[fin] - ref[fin]) <= (beta * scale)[fin]), what


@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("nrhs", [1, 3, 8])
@pytest.mark.parametrize("name", list(CASES))
def test_nonfinite(name, nrhs, store):
    make, srs = CASES[name]
    A = make()
    say("nonfinite", name, nrhs, store)
    rng = np.random.default_rng(17)
    A.vals = np.round(rng.uniform(-1, 1, A.nnz) * 64) / 64  # exact in every storage type; zeros among them
    odd = rng.choice(A.nnz, 4, replace=False)
    A.vals[odd] = [0.0, np.inf, np.nan, np.array(MARK[store], dtype=np.uint64).view(np.float64)]
    shape = (A.n,) if nrhs == 1 else (A.n, nrhs)
    x, g = (np.round(rng.uniform(-1, 1, shape) * 1024) / 1024 for _ in range(2))
    spoil(x, rng)
    spoil(g, rng)
    with np.errstate(invalid="ignore"):
        ref = [OS.spmv(A.row_ptr, A.col_idx, A.vals, x), OA.grad_x(A.row_ptr, A.col_idx, A.vals, g),
               OA.grad_vals(A.row_ptr, A.col_idx, x, g)]
        av, ax, ag = np.abs(A.vals), np.abs(x), np.abs(g)
        scale = [OS.spmv(A.row_ptr, A.col_idx, av, ax), OA.grad_x(A.row_ptr, A.col_idx, av, ag),
                 OA.grad_vals(A.row_ptr, A.col_idx, ax, ag)]
    # one rounding per addition, FP64 or FP32: the longest row or column bounds them all
    most = max(int(np.diff(A.row_ptr).max()), int(np.bincount(A.col_idx).max()), nrhs)
    beta = 1e-12 if store == "f64" else OP.gamma(most, 2.0 ** -24)
    M = CsrkMatrix.from_csr(A.row_ptr, A.col_idx, A.vals, store=store, nrhs=nrhs,
                            params=params(srs, 3, lanes=2, waves=2, reorder="none"))
    B = CsrkBatch([M, M])
    xd, gd = to_dev(x, DT[store]), to_dev(g, DT[store])
    mine = M.values()
    mark = torch.from_numpy(np.array([MARK[store]], dtype=np.uint64).view(np.float64)).to(mine.dtype).cuda()
    if store == "f32":  # the marker's own bits, whatever the conversions above made of its payload
        mark = torch.tensor([0x7FFF0000], dtype=torch.int32).view(torch.float32).cuda()
    if store == "bf16":
        mark = torch.tensor([0x7FFF], dtype=torch.int16).view(torch.bfloat16).cuda()
    mine.view(mark.dtype)[int(odd[3])] = mark[0]
    for vals in (None, mine):
        two = None if vals is None else [vals, vals]
        outs = [(M.spmv(xd, vals=vals),) + M.adjoint(xd, gd, vals=vals)]
        outs += zip(B.spmv([xd, xd], vals=two), *B.adjoint([xd, xd], [gd, gd], vals=two))
        torch.cuda.synchronize()
        for i, out in enumerate(outs):
            for o, r, s, what in zip(out, ref, scale, ("y", "grad_x", "grad_vals")):
                same(o, r, s, beta, f"{what} {'batched' if i else 'alone'} {'handle' if vals is None else 'caller'}")
    B.close()
    M.close()
