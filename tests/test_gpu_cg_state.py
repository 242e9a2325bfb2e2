"""What a CG call leaves behind: x after a breakdown, and the device memory that a handle keeps."""

import numpy as np
import pytest

from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import cg as OCG  # noqa: E402
from paper_2203_05096_amd import _capi as C  # noqa: E402
from paper_2203_05096_amd.matrix import CsrkMatrix  # noqa: E402


def tridiagonal(n, diag, off):
    rp = np.concatenate([[0], np.cumsum(np.r_[2, np.full(n - 2, 3), 2])]).astype(np.int32)
    ci = np.concatenate([[0, 1], (np.arange(1, n - 1)[:, None] + [-1, 0, 1]).ravel(), [n - 2, n - 1]]).astype(np.int32)
    return rp, ci, np.where(ci == np.repeat(np.arange(n), np.diff(rp)), diag, off)


def stream():
    return torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("n", [4099, 500000])
def test_cg_breakdown_leaves_the_updated_x(n, noalloc):
    """A negative definite tridiagonal matrix: p'Ap < 0 at the first iteration, found at the first check.  x is then
    where the iterations so far have taken it, with two launches an iteration (few rows) and with three: the textbook
    iterates in FP64, whose rounding in these few well-conditioned steps is far below the bound."""
    rp, ci, vals = tridiagonal(n, -4.0, 1.0)
    M = CsrkMatrix.from_csr(rp, ci, vals, store="f64")
    perm = M.structure()["perm"]
    b, x0 = np.random.default_rng(8).uniform(-1, 1, (2, n))
    solve = C.csrk_cg_noalloc if noalloc else C.csrk_cg
    for every in (1, 3):
        say("cg breakdown x", n, noalloc, every)
        xd, bd = to_dev(x0[perm], torch.float64), to_dev(b[perm], torch.float64)
        with pytest.raises(C.CsrkError) as e:
            solve(M.handle, bd.data_ptr(), xd.data_ptr(), 1e-12, 50, every, stream())
        assert e.value.name == "CSRK_ERR_UNSUPPORTED"
        ref, it, _ = OCG.cg(rp, ci, vals, b, x0=x0, rtol=1e-12, max_iter=every)
        assert it == every
        x = np.empty(n)
        x[perm] = xd.cpu().numpy()
        assert np.max(np.abs(x - ref)) <= 1e-12 * np.max(np.abs(ref))
    M.close()


def test_cg_memory_a_handle_keeps():
    """A handle keeps the work vectors of its last solve up to CSRK_CG_NOALLOC_BYTES, gives them back when asked and
    takes new ones for the next; a larger solve's are freed when the call returns."""
    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    page = 2 << 20  # what the allocator rounds a block to
    for n in (4099, 3000000, 2000000, 300000):  # the first one loads the kernels
        rp, ci, vals = tridiagonal(n, 4.0, -1.0)
        M, M2 = (CsrkMatrix.from_csr(rp, ci, vals, store="f64") for _ in range(2))
        M.cg_release()  # nothing kept yet
        b = torch.ones(n, dtype=torch.float64, device="cuda")
        xs = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(3)]

        def solve(x, M=M):
            return C.csrk_cg(M.handle, b.data_ptr(), x.data_ptr(), 1e-9, 50, 5, stream())
        need = C.csrk_cg_noalloc_bytes(M.handle)
        start = free()
        first = solve(xs[0])
        held = start - free()
        again, at_rest = solve(xs[1]), start - free()
        M.cg_release()
        # the runtime keeps small blocks that are freed for the next that asks: another handle's solve takes this one
        other, reused = solve(xs[2], M2), start - free()
        M2.cg_release()
        say("cg memory", n, need, held, at_rest, reused)
        if n > 4099:
            if need > C.CG_NOALLOC_BYTES:
                assert held <= page and at_rest <= page
            else:
                assert need - page <= held <= need + 2 * page and abs(at_rest - held) <= page
            assert reused <= held + page
        assert first == again == other and torch.equal(xs[0], xs[1]) and torch.equal(xs[0], xs[2])
        xs[2].zero_()
        assert solve(xs[2]) == first and torch.equal(xs[0], xs[2])  # with new work memory
        M.close()
        M2.close()
    with pytest.raises(C.CsrkError) as e:
        C.csrk_cg_release(None)
    assert e.value.name == "CSRK_ERR_ARG"
