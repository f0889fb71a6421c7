"""Applications, diagonals, gradients and misfits on numberings that scatter an
element's nodes over memory (random ids, and nodes ordered by vertices, edges,
faces and interiors), at sizes on both sides of those from which the calls go
through the internal order, against an operator of the same mesh that keeps the
caller's order and so never does. Bar: 1e-12 normwise in FP64, 2e-6 in FP32 (as
against the oracle in the parity tests)."""
import numpy as np
import pytest

import synth
import paper_2004_06722_amd.bp as B
from tests.gpu_cases import rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def renumbered(m, kind, p):
    rng = np.random.default_rng(61)
    if kind == "random":
        new = rng.permutation(m.nglobal)
    else:
        edge = [np.arange(p * n + 1) % p == 0 for n in (m.ez, m.ey, m.ex)]
        on = (edge[0][:, None, None].astype(int) + edge[1][None, :, None]
              + edge[2][None, None, :]).ravel()
        new = np.empty(m.nglobal, dtype=np.int64)
        new[np.argsort(-on, kind="stable")] = np.arange(m.nglobal)
    boundary = np.empty_like(m.boundary)
    boundary[new] = m.boundary
    return new[m.elem_dofs], boundary


@pytest.mark.parametrize("bp,p,e,ncomp,kind", [
    (5, 2, 22, 1, "random"), (5, 3, 26, 3, "random"), (5, 4, 20, 1, "random"),
    (5, 7, 12, 1, "random"), (6, 5, 16, 2, "random"), (5, 6, 14, 1, "entities"),
    (5, 8, 11, 1, "entities"), (3, 2, 30, 2, "random"), (3, 5, 17, 1, "random"),
    (4, 4, 20, 3, "random"), (3, 7, 12, 1, "entities")])
def test_both_routes_agree(bp, p, e, ncomp, kind):
    q, quad = B.bp_quadrature(bp, p)
    xi, _ = B.rule(p + 1, B.GLL)
    m = synth.brick_mesh(e, e, e, p, xi, seed=62)
    dofs, boundary = renumbered(m, kind, p)
    n = m.nglobal
    shape = (n,) if ncomp == 1 else (ncomp, n)
    gen = torch.Generator(device="cuda").manual_seed(63)
    u = torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
    v = torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
    kappa = 0.5 + torch.rand((dofs.shape[0], q ** 3), dtype=torch.float64, device="cuda",
                             generator=gen)

    def results(caller_order):
        out = {}
        with B.Operator(p, q, quad, dofs, m.node_xyz, n, boundary, ncomp=ncomp, fp32=True,
                        caller_order=caller_order) as op:
            op.set_coeff(kappa)
            op.set_helmholtz(3.0)
            for which in (B.MASS, B.STIFF, B.HELM):
                for masked in (False, True):
                    out[which, masked] = op.apply(which, u, masked=masked)
                    out[which, masked, "32"] = op.apply(which, u.float(), masked=masked)
                    out[which, masked, "diag"] = op.diag(which, masked=masked)
            out["misfit"], out["gradient"] = op.mass_misfit(u, v)
            assert op.mass_misfit(u, v, grad=False)[0] == out["misfit"]
            if quad == B.GLL:
                out["kappa"] = op.grad_kappa(u, v)
            torch.cuda.synchronize()
            return {k: x if isinstance(x, float) else x.cpu().numpy() for k, x in out.items()}

    ref, got = results(True), results(False)
    for k in ref:
        assert rel(got[k], ref[k]) <= (2e-6 if "32" in str(k) else 1e-12), k
