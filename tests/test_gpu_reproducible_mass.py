"""The assembled mass matrix of a collocated operator, a diagonal, is the same
in every bit for every operator built on the same mesh, and with it the misfit's
loss and gradient and the mass application: the order in which work-groups
arrive plays no part. Each entry is the sum of the node's B~ rounded once."""
import numpy as np
import pytest

import synth
import paper_2004_06722_amd.bp as B
from oracle.operators import MASS
from tests.gpu_cases import TOL, Case, rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p,grid,caller_order", [(1, (24, 24, 24), False), (2, (16, 16, 16), False),
                                                 (3, (12, 12, 12), True), (7, (5, 5, 5), False)])
def test_every_set_up_gives_the_same_bits(p, grid, caller_order):
    xi, _ = B.rule(p + 1, B.GLL)
    m = synth.scramble_mesh(synth.brick_mesh(*grid, p, xi, seed=3), 5)
    rng = np.random.default_rng(11)
    u = torch.tensor(rng.standard_normal(m.nglobal), device="cuda")
    ut = torch.tensor(rng.standard_normal(m.nglobal), device="cuda")
    seen = set()
    for _ in range(8):
        with B.Operator(p, p + 1, B.GLL, m.elem_dofs, m.node_xyz, m.nglobal, None,
                        caller_order=caller_order) as op:
            loss, grad = op.mass_misfit(u, ut)
            w = op.apply(MASS, u, masked=False)
            torch.cuda.synchronize()
            seen.add((loss, grad.cpu().numpy().tobytes(), w.cpu().numpy().tobytes()))
    assert len(seen) == 1


@pytest.mark.parametrize("ncomp", [1, 3])
def test_nodes_of_many_slots_and_of_none(ncomp):
    # random ids over a sixtieth of the slots, two ids that no element names,
    # and element sizes that span twelve orders of magnitude in volume: a
    # node's terms reach from the largest to far below its last bit
    p = 2
    c = Case(5, p, 4, 4, 4, seed=13, ncomp=ncomp, dirichlet=False)
    try:
        xi, _ = B.rule(p + 1, B.GLL)
        m = synth.brick_mesh(4, 4, 4, p, xi, seed=13)
        rng = np.random.default_rng(14)
        n = m.elem_dofs.size // 60
        dofs = rng.integers(0, n, size=m.elem_dofs.shape)
        size = 10.0 ** rng.uniform(-4, 0, size=(m.elem_dofs.shape[0], 1, 1))
        u = rng.standard_normal((ncomp, n + 2))
        with B.Operator(p, p + 1, B.GLL, dofs, m.node_xyz * size, n + 2, ncomp=ncomp) as op:
            ones = torch.ones((ncomp, n + 2), dtype=torch.float64, device="cuda")
            md = op.apply(MASS, ones, masked=False).cpu().numpy()[0]
            # B_L 1 of every element alone, summed on the host
            bl = op.apply_local(MASS, torch.ones((ncomp, dofs.size), dtype=torch.float64,
                                                 device="cuda")).cpu().numpy()[0]
            ref = np.zeros(n + 2, dtype=np.longdouble)
            np.add.at(ref, dofs.ravel(), bl.astype(np.longdouble))
            assert np.all(md[n:] == 0.0)
            assert np.all(np.abs(md - ref.astype(np.float64)) <= np.spacing(md))
            w = op.apply(MASS, torch.tensor(u, device="cuda"), masked=False).cpu().numpy()
            assert rel(w, md * u) <= TOL
    finally:
        c.close()


@pytest.mark.parametrize("p,grid", [(1, (3, 2, 5)), (5, (13, 12, 12)), (7, (5, 5, 5))])
def test_diagonal_is_the_assembled_matrix(p, grid):
    # bp_diag gives the entries that an application multiplies by, bit for bit, 0
    # on masked nodes and on those of no element
    xi, _ = B.rule(p + 1, B.GLL)
    m = synth.scramble_mesh(synth.brick_mesh(*grid, p, xi, seed=3), 5)
    bd = np.concatenate([np.asarray(m.boundary, dtype=bool), [False]])
    with B.Operator(p, p + 1, B.GLL, m.elem_dofs, m.node_xyz, m.nglobal + 1, bd) as op:
        ones = torch.ones(m.nglobal + 1, dtype=torch.float64, device="cuda")
        for masked in (False, True):
            d = op.diag(MASS, masked=masked).cpu().numpy()
            assert np.array_equal(d, op.apply(MASS, ones, masked=masked).cpu().numpy())
            assert np.array_equal(d == 0.0, bd & masked | (np.arange(d.size) == m.nglobal))
