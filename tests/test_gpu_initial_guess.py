"""A guess that is zero all but one entry: the pass that looks for a non-zero
entry decides whether A x0 is subtracted at all, so one entry that it misses
gives a wrong residual. The entry lies first, last, in the last component alone,
and around each bound of that pass (256 threads a work-group, 2048 work-groups,
four entries a thread and round, one by one in the remainder). The solve from
x0 must give x0 + y with y the solve of b - A x0 from zero, whose guess has
nothing to find: the same recurrences on the same residual. Bar: normwise 1e-12;
the entry is such that missing it changes the result by its own size."""
import numpy as np
import pytest

from oracle.operators import MASS, STIFF
from oracle.pcg import pcg
from paper_2004_06722_amd import BpError
from tests.gpu_cases import TOL, Case, rel
from tests.test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROUND = 2048 * 256


@pytest.mark.parametrize("caller_order", [False, True])
@pytest.mark.parametrize("sr", [False, True])
@pytest.mark.parametrize("bp,p,ncomp", [(5, 3, 1), (6, 2, 3), (1, 3, 1), (4, 2, 2)])
def test_one_entry_against_the_oracle(bp, p, ncomp, sr, caller_order):
    c = Case(bp, p, 3, 3, 2, seed=50 + p, ncomp=ncomp, caller_order=caller_order)
    try:
        c.op.set_cg_variant(sr)
        which, masked = (MASS, False) if bp == 1 else (STIFF, True)
        mask = np.ones(c.disc.nglobal) if bp == 1 else 1.0 - c.mesh.boundary
        free = np.flatnonzero(mask)
        b = c.vec(51) * (mask[:, None] if ncomp > 1 else mask)
        for node, comp in ((free[0], 0), (free[-1], 0), (free[0], ncomp - 1),
                           (free[-1], ncomp - 1), (free[len(free) // 2], ncomp // 2)):
            x0 = np.zeros_like(b)
            if ncomp > 1:
                x0[node, comp] = 3.0
            else:
                x0[node] = 3.0
            rec = []
            pcg(lambda v: c.disc.apply(which, v, masked=masked), b,
                c.disc.jacobi_inverse(which, masked=masked), x0=x0, maxit=4, fixed_iters=True,
                record=rec)
            for k in (1, 4):
                x, _ = c.op.pcg_solve(dev(b), x=dev(x0), which=which, maxit=k, fixed_iters=True)
                assert rel(host(x), rec[k - 1]) <= TOL, (node, comp, k)
            x0[x0 != 0] = np.nan
            with pytest.raises(BpError, match="BP_ERR_NONFINITE"):
                c.op.pcg_solve(dev(b), x=dev(x0), which=which, maxit=4, fixed_iters=True)
    finally:
        c.close()


@pytest.mark.parametrize("bp,p,grid,ncomp", [(5, 3, (44, 44, 44), 1), (6, 2, (44, 44, 44), 3),
                                             (1, 3, (44, 44, 44), 1)])
def test_one_entry_around_the_rounds_of_the_pass(bp, p, grid, ncomp):
    # 2.35e6 entries (one whole round of four entries a thread and a remainder
    # in single ones) and three times 7.05e5
    c = Case(bp, p, *grid, seed=None, ncomp=ncomp)
    try:
        which, masked = (MASS, False) if bp == 1 else (STIFF, True)
        n = c.disc.nglobal
        free = np.ones(n, bool) if bp == 1 else c.mesh.boundary == 0
        rng = np.random.default_rng(52)
        shape = (n,) if ncomp == 1 else (ncomp, n)
        b = torch.tensor(rng.standard_normal(shape) * free, device="cuda")
        for at in (0, 255, 256, ROUND - 1, ROUND, 2 * ROUND, 3 * ROUND + 1, 4 * ROUND - 1, 4 * ROUND,
                   4 * ROUND + 256, n * ncomp - 1):
            if at >= n * ncomp:
                continue
            # the nearest free node at or after it (before it at the end)
            flat = np.tile(free, ncomp)
            after = np.flatnonzero(flat[at:at + 200000])
            at = at + after[0] if after.size else np.flatnonzero(flat[:at])[-1]
            x0 = torch.zeros_like(b)
            x0.view(-1)[int(at)] = 1e3
            r0 = b - c.op.apply(which, x0, masked=masked)
            for sr in (False, True):
                c.op.set_cg_variant(sr)
                y, _ = c.op.pcg_solve(r0, which=which, maxit=3, fixed_iters=True)
                x, _ = c.op.pcg_solve(b, x=x0.clone(), which=which, maxit=3, fixed_iters=True)
                torch.cuda.synchronize()
                assert float(torch.norm(x - (x0 + y)) / torch.norm(x)) <= TOL, (at, sr)
    finally:
        c.close()
