"""An NMF of few ranks over many rows goes to the kernel with a row a thread, and to the matrix cores when
its launch holds a problem of more ranks: the same bits, either side of each line."""
import pytest
import torch

import paper_1909_07570_amd as nnc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,m", [(128, 8, 4), (129, 3, 4), (512, 16, 1), (200, 17, 4), (300, 8, 5), (420, 2, 6),
                                         (300, 9, 6), (257, 8, 7)])
def test_same_bits_in_either_kernel(rows, cols, m):
    gen = torch.Generator().manual_seed(rows + cols + m)
    u = lambda *s: torch.rand(*s, generator=gen) + 1e-2
    a, w0, h0 = u(rows, cols).cuda(), u(rows, m).cuda(), u(m, cols).cuda()
    w0[5] = 0.0  # clipped denominators
    w, h = w0.clone(), h0.clone()
    res = nnc.nmf_fit(a, m, 30, w, h)
    other = [u(20, cols).cuda(), u(20, 9).cuda(), u(9, cols).cuda()]
    w2, h2 = w0.clone(), h0.clone()
    both = nnc.nmf_fit_batched([a, other[0]], [m, 9], 30, [w2, other[1]], [h2, other[2]])
    assert torch.equal(w, w2) and torch.equal(h, h2)
    assert abs(float(res) - float(both[0])) <= 1e-12 * float(res)
