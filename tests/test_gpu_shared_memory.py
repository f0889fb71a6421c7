"""Results that share memory with inputs: windows of one buffer, the result's
shifted against the input's by one entry, by a few elements' nodes or by half its
length. Each entry point reads its whole input before it overwrites any of it:
the results are those of separate buffers. Bar: 1e-13 normwise (the order of at
most eight additions a node differs)."""
import ctypes

import numpy as np
import pytest

from oracle.operators import MASS, STIFF
from paper_2004_06722_amd import _lib
from tests.gpu_cases import Case, rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def window(buffer, at, count):
    return buffer[at:at + count], ctypes.c_void_p(buffer.data_ptr() + 8 * at)


@pytest.mark.parametrize("bp,p,grid,ncomp", [(5, 7, (12, 12, 12), 1), (6, 3, (16, 16, 16), 3),
                                             (3, 5, (10, 10, 10), 1)])
def test_windows_of_one_buffer(bp, p, grid, ncomp):
    lib = _lib.load()
    c = Case(bp, p, *grid, seed=30, ncomp=ncomp)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    try:
        nv, ng = c.disc.nglobal * ncomp, c.disc.E * c.q ** 3
        shape = (c.disc.nglobal,) if ncomp == 1 else (ncomp, c.disc.nglobal)
        rng = np.random.default_rng(31)
        u = torch.tensor(rng.standard_normal(shape), device="cuda")
        v = torch.tensor(rng.standard_normal(shape), device="cuda")
        buffer = torch.empty(4 * max(nv, ng), dtype=torch.float64, device="cuda")
        grad = c.quad == _lib.BP_QUAD_GLL
        ref = {w: c.op.apply(w, u, masked=True).cpu().numpy().ravel() for w in (MASS, STIFF)}
        loss, dv = c.op.mass_misfit(u, v)
        g = c.op.grad_kappa(u, v).cpu().numpy().ravel() if grad else None
        for shift in (1, 3 * (p + 1) ** 3, nv // 2):
            for first, second in ((0, shift), (shift, 0)):
                for which in (MASS, STIFF):
                    uw, up = window(buffer, first, nv)
                    ww, wp = window(buffer, second, nv)
                    uw.copy_(u.view(-1))
                    assert lib.bp_apply(c.op._h, which, _lib.BP_FP64, up, wp, _lib.BP_MASKED,
                                        stream) == 0
                    torch.cuda.synchronize()
                    assert rel(ww.cpu().numpy(), ref[which]) <= 1e-13, (which, shift)
                for mine, other in ((u, v), (v, u)):
                    uw, up = window(buffer, first, nv)
                    ww, wp = window(buffer, second, nv)
                    uw.copy_(mine.view(-1))
                    op = ctypes.c_void_p(other.data_ptr())
                    a, b = (up, op) if mine is u else (op, up)
                    out = ctypes.c_double()
                    assert lib.bp_mass_misfit(c.op._h, a, b, wp, ctypes.byref(out), stream) == 0
                    assert out.value == loss
                    assert rel(ww.cpu().numpy(), dv.cpu().numpy().ravel()) <= 1e-13, shift
                    if not grad:
                        continue
                    uw.copy_(mine.view(-1))
                    gw, gp = window(buffer, second, ng)
                    a, b = (up, op) if mine is u else (op, up)
                    assert lib.bp_grad_kappa(c.op._h, a, b, gp, stream) == 0
                    torch.cuda.synchronize()
                    assert rel(gw.cpu().numpy(), g) <= 1e-13, shift
    finally:
        c.close()
