"""Work-groups taken in runs per XCD: meshes whose operators have just fewer
than, exactly and just more than one or two whole rounds of 8 x 32 (8 x 16 for
the Gauss-Legendre stiffness) work-groups, and none. At p = 7 the collocated
kernel has one element per work-group, the Gauss-Legendre kernels three; a
group taken twice or left out shows in the assembled apply, a misplaced partial
row in the iterates. The reference is w = Q^T A_L Q u from the element-local
apply, whose work-groups keep the launch order, with the gather and the sums on
the host, and the oracle's PCG on it. (The oracle's own factors come from nodes
1.1e-16 apart from the library's; on a mesh of 513 elements along one axis that
alone moves A u by 1.0e-12.) Bar: normwise 1e-12, as in the parity tests."""
import numpy as np
import pytest

from oracle.operators import MASS, STIFF
from oracle.pcg import pcg
from tests.gpu_cases import TOL, Case, rel
from tests.test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bp,grid", [(5, (17, 15, 1)), (5, (16, 16, 1)), (5, (257, 1, 1)),
                                     (5, (513, 1, 1)), (3, (127, 3, 1)), (3, (32, 12, 1)),
                                     (3, (55, 7, 1)), (1, (51, 15, 1)), (1, (32, 24, 1)),
                                     (1, (257, 3, 1)), (1, (2, 2, 1))])
def test_apply_and_iterates_around_whole_rounds_of_work_groups(bp, grid):
    which = MASS if bp == 1 else STIFF
    c = Case(bp, 7, *grid, seed=bp)
    try:
        dofs = np.asarray(c.mesh.elem_dofs)
        free = np.ones(c.disc.nglobal) if c.dir is None else 1.0 - np.asarray(c.dir)

        def apply(v, masked):
            m = free if masked else 1.0
            wl = host(c.op.apply_local(which, dev((m * v)[dofs].ravel())))
            return m * np.bincount(dofs.ravel(), weights=wl, minlength=c.disc.nglobal)

        u = c.vec(31)
        assert rel(host(c.op.apply(which, dev(u), masked=False)), apply(u, False)) <= TOL
        b = c.vec(32) * free
        d = host(c.op.diag(which, masked=bp > 1))
        rec = []
        pcg(lambda v: apply(v, bp > 1), b, np.where(d != 0, 1 / np.where(d != 0, d, 1), 0),
            maxit=2, fixed_iters=True, record=rec)
        x, _ = c.op.pcg_solve(dev(b), which=which, maxit=2, fixed_iters=True)
        assert rel(host(x), rec[-1]) <= TOL
    finally:
        c.close()
