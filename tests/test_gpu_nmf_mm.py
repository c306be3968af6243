"""The NMF sweeps on the matrix cores at the edges of their tiles, forms and LDS layout."""
import pytest
import torch

import paper_1909_07570_amd as nnc

pytestmark = pytest.mark.gpu
EPS = 1e-12
SWEEPS = 4


def _nmf64(a, w, h):
    for _ in range(SWEEPS):
        w = w * (a @ h.T) / (w @ (h @ h.T)).clamp_min(EPS)
        h = h * (w.T @ a) / ((w.T @ w) @ h).clamp_min(EPS)
    return w, h


@pytest.mark.parametrize(
    "rows,cols,ranks",
    [
        ((1, 3, 16), 1, (1, 1, 1)),  # fewer rows than row ranges, one column
        ((17, 31, 64), 4, (3, 4, 5)),  # a last tile of one row; ranks at a quad
        ((15, 130, 33), 8, (16, 15, 9)),  # full tiles of ranks
        ((40, 512, 77), 10, (17, 20, 3)),  # ranks of the tail quad, and none
        ((63, 200, 96), 12, (18, 19, 20)),
        ((100, 50, 31), 13, (21, 24, 2)),  # two and a half tiles of ranks
        ((64, 90, 48), 17, (25, 32, 16)),
        ((70, 33, 20), 32, (32, 1, 17)),
        ((512, 481, 500), 16, (20, 17, 20)),  # largest padded layout
        ((2000, 40, 9), 8, (4, 4, 4)),  # padded layout does not fit
    ],
)
def test_sweeps(rows, cols, ranks):
    gen = torch.Generator().manual_seed(sum(rows) + cols)
    a = [torch.rand(n, cols, generator=gen) + 1e-2 for n in rows]
    w = [torch.rand(n, m, generator=gen) + 1e-2 for n, m in zip(rows, ranks)]
    h = [torch.rand(m, cols, generator=gen) + 1e-2 for m in ranks]
    for x in w:
        if len(x) > 3:
            x[3] = 0.0  # clipped denominators: the row stays zero
    wg, hg = [x.cuda() for x in w], [x.cuda() for x in h]
    res = nnc.nmf_fit_batched([x.cuda() for x in a], list(ranks), SWEEPS, wg, hg)
    # A chain of n products is off by at most n 2^-24; a sweep has chains over the columns, the ranks and
    # (ranges of at most 64 rows and 32 ranges) the rows in W and then H, and its quotients pass on what the
    # sweeps before were off by, at most doubled.
    tol = 2.0 ** -24 * (2 * cols + 2 * max(ranks) + 2 * 96) * (2 ** SWEEPS - 1)
    for k in range(len(rows)):
        ew, eh = _nmf64(a[k].double(), w[k].double(), h[k].double())
        for got, want in ((wg[k], ew), (hg[k], eh)):
            assert (got.double().cpu() - want).norm() <= tol * want.norm()
        rel = (a[k].double() - wg[k].double().cpu() @ hg[k].double().cpu()).norm() / a[k].double().norm()
        # the residual is that of the W H of the result, its products in FP32
        assert abs(float(res[k]) - float(rel)) <= 2.0 ** -24 * (max(ranks) + 2) * 4
