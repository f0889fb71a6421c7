"""Solves on both sides of the bounds that choose how an iteration is launched.
How partial tables are folded: above 16384 rows, or 32768 sums. How many launches
it takes: vector rows per thread of the operator's work-groups (20 in FP64: p = 7
between E = 15^3 and 16^3; p = 3 with 14, p = 4 with 12). The
iterates of every form are those of the five launches, normwise to 1e-12."""
import pytest

import synth
import paper_2004_06722_amd.bp as B
from paper_2004_06722_amd import _lib
from tests.gpu_cases import TOL

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def operator(p, grid, ncomp=1):
    xi, _ = B.rule(p + 1, B.GLL)
    m = synth.brick_mesh(*grid, p, xi, seed=6)
    op = B.Operator(p, p + 1, B.GLL, m.elem_dofs, m.node_xyz, m.nglobal, m.boundary, ncomp=ncomp)
    gen = torch.Generator(device="cuda").manual_seed(7)
    shape = (m.nglobal,) if ncomp == 1 else (ncomp, m.nglobal)
    b = torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
    return op, b * torch.tensor(1.0 - m.boundary, device="cuda")


@pytest.mark.parametrize("p,grid", [(7, (15, 15, 15)), (7, (16, 15, 16)), (7, (16, 16, 16)),
                                    (3, (32, 32, 32)), (4, (29, 28, 28))])
def test_iterates_on_both_sides(p, grid):
    op, b = operator(p, grid)
    with op:
        ref = {}
        for fuse in (0, 2):
            op.set_option(_lib.BP_OPT_CG_FUSE, fuse)
            for iters in (1, 5):
                x, st = op.pcg_solve(b, maxit=iters, fixed_iters=True)
                torch.cuda.synchronize()
                assert st["iters"] == iters
                ref.setdefault(iters, x)
                err = float(torch.norm(x - ref[iters]) / torch.norm(ref[iters]))
                assert err <= TOL, (fuse, iters, err)


@pytest.mark.parametrize("p,grid,ncomp", [(7, (32, 32, 16), 1), (7, (32, 32, 17), 1),
                                          (7, (32, 32, 16), 2), (7, (33, 16, 16), 4),
                                          (7, (32, 16, 16), 4)])
def test_folded_and_direct_sums_agree(p, grid, ncomp):
    # one work-group an element at p = 7: operator tables of 16384 and 17408 rows of
    # one sum, 16384 of two, 8448 and 8192 of four. The two- or four-launch and the
    # five-launch forms sum tables of other lengths
    op, b = operator(p, grid, ncomp)
    with op:
        ref = None
        for fuse, sr in ((0, False), (2, False), (0, True)):
            op.set_option(_lib.BP_OPT_CG_FUSE, fuse)
            op.set_cg_variant(sr)
            x, _ = op.pcg_solve(b, maxit=4, fixed_iters=True)
            torch.cuda.synchronize()
            ref = x if ref is None else ref
            assert float(torch.norm(x - ref) / torch.norm(ref)) <= TOL, (fuse, sr)
            # the residual that the sums give is the true one
            r = b - op.apply(B.STIFF, x)
            _, st = op.pcg_solve(b, x=x.clone(), maxit=0)
            true = float(torch.norm(r) / torch.norm(b)) if ncomp == 1 else float(
                torch.norm(r[0]) / torch.norm(b[0]))
            assert abs(st["rel_res"][0] - true) <= 1e-12 * max(true, 1.0)
