"""The scaled factors kappa G of every form of their kernel -- elements of fewer
than 64 points (p = 1, 2, and p = 1 on Gauss points), one point per thread, and that
with streaming access (G of 128 MiB and more) -- through the operator they enter:
A(kappa) u with kappa constant per element must equal the sum over the elements of
kappa_e times their own A^e u, from the element-local operator without a
coefficient. FP64 to 1e-13 normwise (a product rounded in another place), FP32 to
2e-6. Then kappa varying inside the elements against the transposed product with
kappa = 1: u^T A(kappa) u = sum kappa_q (Du)^T G (Du), linear in kappa."""
import pytest

import synth
import paper_2004_06722_amd.bp as B

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bp,p,e", [(5, 1, 7), (5, 2, 6), (5, 3, 5), (5, 4, 4), (5, 6, 21),
                                    (3, 1, 7), (3, 2, 5), (3, 3, 29), (3, 4, 24), (3, 6, 3)])
def test_scaled_factors(bp, p, e):
    q, quad = B.bp_quadrature(bp, p)
    xi, _ = B.rule(p + 1, B.GLL)
    m = synth.brick_mesh(e, e, e, p, xi, seed=71)
    E, n3 = m.elem_dofs.shape
    gen = torch.Generator(device="cuda").manual_seed(72)
    uL = torch.randn((E, n3), dtype=torch.float64, device="cuda", generator=gen)
    ke = 0.5 + torch.rand((E, 1), dtype=torch.float64, device="cuda", generator=gen)
    kq = 0.5 + torch.rand((2, E, q ** 3), dtype=torch.float64, device="cuda", generator=gen)
    with B.Operator(p, q, quad, m.elem_dofs, m.node_xyz, m.nglobal, m.boundary,
                    fp32=True) as op:
        plain = op.apply_local(B.STIFF, uL)
        plain32 = op.apply_local(B.STIFF, uL.float())
        op.set_coeff((ke * torch.ones((E, q ** 3), dtype=torch.float64,
                                      device="cuda")).contiguous())
        for got, ref, tol in ((op.apply_local(B.STIFF, uL), ke * plain, 1e-13),
                              (op.apply_local(B.STIFF, uL.float()).double(),
                               ke * plain32.double(), 2e-6)):
            assert float(torch.norm(got - ref) / torch.norm(ref)) <= tol
        # linear in kappa, point by point
        parts = []
        for k in (kq[0], kq[1], kq[0] + 2.0 * kq[1]):
            op.set_coeff(k.contiguous())
            parts.append(op.apply_local(B.STIFF, uL))
        ref = parts[0] + 2.0 * parts[1]
        assert float(torch.norm(parts[2] - ref) / torch.norm(ref)) <= 1e-13
        # one point's kappa reaches that point alone: the element's energy moves by
        # its own term, the same whether the other points have kappa 1 or 2
        one = torch.ones((E, q ** 3), dtype=torch.float64, device="cuda")
        point = q ** 3 // 3
        terms = []
        for base in (1.0, 2.0):
            energies = []
            for extra in (0.0, 1.0):
                k = base * one
                k[:, point] += extra
                op.set_coeff(k)
                energies.append((uL * op.apply_local(B.STIFF, uL)).sum(1))
            terms.append(energies[1] - energies[0])
        scale = float((uL * plain).sum(1).abs().max())
        assert float((terms[0] - terms[1]).abs().max()) <= 1e-12 * scale
        assert float(terms[0].min()) > 0.0
