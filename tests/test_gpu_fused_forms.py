"""The fused CG iterations (two and three launches) beyond their small-mesh
sizes and in FP32: four nodes per thread in the vector kernels, several
components, the tables of more than 1024 groups, and the FP32 inner solves of
both mixed modes (the reliable one resumes a fused iteration after every
replacement). Against the five-launch iteration, BP_OPT_CG_FUSE = 0."""
import numpy as np
import pytest

import synth
from oracle.operators import MASS, STIFF
from paper_2004_06722_amd import _lib
from tests.gpu_cases import TOL, Case, rel
from tests.test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bp,p,grid,ncomp", [(3, 7, (10, 10, 9), 1), (4, 5, (14, 14, 14), 3),
                                             (6, 9, (8, 8, 7), 4), (5, 10, (7, 7, 6), 1),
                                             (6, 7, (6, 6, 5), 5), (5, 7, (15, 15, 14), 1)])
def test_iterates_match_the_five_launch_form(bp, p, grid, ncomp):
    c = Case(bp, p, *grid, seed=p, ncomp=ncomp)
    try:
        mask = 1 - c.mesh.boundary
        b = c.vec(5) * (mask[:, None] if ncomp > 1 else mask)
        ref = {}
        for fuse in (0, 1, 2):
            c.op.set_option(_lib.BP_OPT_CG_FUSE, fuse)
            for iters in (1, 6):
                x, st = c.op.pcg_solve(dev(b), which=STIFF, maxit=iters, fixed_iters=True)
                assert st["iters"] == iters
                x = host(x)
                if fuse == 0:
                    ref[iters] = x
                assert rel(x, ref[iters]) <= TOL, (fuse, iters)
    finally:
        c.close()


@pytest.mark.parametrize("p,grid,ncomp", [(2, (3, 3, 2), 1), (7, (3, 3, 3), 1), (7, (9, 9, 9), 1),
                                          (5, (4, 3, 3), 3), (10, (2, 2, 2), 1)])
@pytest.mark.parametrize("reliable", [False, True])
def test_fp32_inner_solves(p, grid, ncomp, reliable):
    c = Case(5, p, *grid, seed=p, ncomp=ncomp, fp32=True)
    try:
        f = synth.manufactured_f(c.mesh.global_coords())
        b = c.disc.apply(MASS, f, masked=False) * c.disc.mask
        if ncomp > 1:
            b = np.stack([b * (k + 1) for k in range(ncomp)], axis=1)
        counts = []
        for fuse in (0, 1, 2, 3):
            c.op.set_option(_lib.BP_OPT_CG_FUSE, fuse)
            x, st = c.op.pcg_solve_mixed(dev(b), outer_rtol=1e-10, inner_rtol=1e-1 if reliable
                                         else 1e-4, max_outer=200, max_inner=20000,
                                         reliable=reliable)
            r = b - c.disc.apply(STIFF, host(x))
            assert st["converged"] and np.linalg.norm(r) / np.linalg.norm(b) <= 1.2e-10, fuse
            counts.append(st["iters"])
        # the same recurrences: rounding alone may move the count
        assert max(counts) <= 1.25 * min(counts) + 5, counts
    finally:
        c.close()
