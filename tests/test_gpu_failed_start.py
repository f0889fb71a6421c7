"""A solve that cannot be started returns its error and leaves x as the caller
gave it, whatever the solves before it left in the operator's buffers. The
failure is an error code that an earlier HIP call of the caller's own has left
behind: the library's first launch check collects it and ends the solve before
its initialisation."""
import ctypes
import re

import numpy as np
import pytest

from oracle.operators import MASS, STIFF
from paper_2004_06722_amd import _lib
from tests.gpu_cases import Case
from tests.test_gpu_parity import dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def leave_an_error_behind():
    """A device index beyond the last, which the runtime refuses."""
    path = re.search(r"\S*/libamdhip64\.so\S*", open("/proc/self/maps").read()).group(0)
    assert ctypes.CDLL(path).hipSetDevice(1 << 20) != 0


@pytest.mark.parametrize("guess", ["zero", "one entry"])
@pytest.mark.parametrize("entry,sr", [("bp_pcg_solve", False), ("bp_pcg_solve", True),
                                      ("bp_pcg_solve_static", False)])
@pytest.mark.parametrize("bp,ncomp,caller_order", [(5, 1, False), (6, 3, False), (1, 1, False),
                                                   (5, 1, True)])
def test_x_is_left_as_given(bp, ncomp, caller_order, entry, sr, guess):
    c = Case(bp, 4, 3, 2, 2, seed=9, ncomp=ncomp, caller_order=caller_order)
    try:
        c.op.set_cg_variant(sr)
        which = MASS if bp == 1 else STIFF
        b = dev(c.vec(10))
        start = torch.zeros_like(b)
        if guess == "one entry":
            start.view(-1)[c.disc.nglobal // 2] = 1.5
        solve = getattr(_lib.load(), entry)
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

        def run(x):
            return solve(c.op._h, which, ctypes.c_void_p(b.data_ptr()),
                         ctypes.c_void_p(x.data_ptr()), 0.0, 4, 1, None, stream)

        x = start.clone()
        assert run(x) == 0                       # leaves a solution in the buffers
        first = x.clone()
        x = start.clone()
        torch.cuda.synchronize()
        leave_an_error_behind()
        assert run(x) == _lib.BP_ERR_HIP
        torch.cuda.synchronize()
        assert torch.equal(x, start)
        assert run(x) == 0                       # and the operator is as good as before
        assert np.linalg.norm((x - first).cpu().numpy()) <= 1e-12 * float(torch.norm(first))
    finally:
        c.close()
