"""Device memory that an operator takes: the arrays that its entry points need
and no more. Collocated operators in the internal order with FP32 data: two
gather maps, two permutations, the factors and the diagonals in their precisions,
and as vectors r, p, w, the scratch vector and x in FP64, r, p, w, x and b in
FP32. Allowed over the sum: 2 MiB an array (the driver's page)."""
import gc

import pytest

import synth
import paper_2004_06722_amd.bp as B

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("ncomp,fp32", [(1, False), (1, True), (3, True)])
def test_set_up_takes_the_sum_of_its_arrays(ncomp, fp32):
    p, e = 4, 56
    xi, _ = B.rule(p + 1, B.GLL)
    m = synth.brick_mesh(e, e, e, p, xi, seed=None)
    n, nl = m.nglobal, m.elem_dofs.size
    args = (p, p + 1, B.GLL, m.elem_dofs, m.node_xyz, n, m.boundary)
    with B.Operator(*args, ncomp=ncomp, fp32=fp32) as op:   # the runtime's own first allocations
        torch.cuda.synchronize()
    gc.collect()
    before = free_bytes()
    with B.Operator(*args, ncomp=ncomp, fp32=fp32) as op:
        used = before - free_bytes()
    arrays = [(2, 4 * nl), (2, 4 * n), (1, 8 * 7 * nl), (3, 8 * n), (5, 8 * n * ncomp)]
    if fp32:
        arrays += [(1, 4 * 7 * nl), (1, 4 * n), (5, 4 * n * ncomp)]
    total = sum(k * b for k, b in arrays)
    # the arrays above and no more than eight small ones
    count = sum(k for k, _ in arrays) + 8
    assert used <= total + count * (1 << 21), (used, total)
