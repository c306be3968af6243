"""CP of the data tensor: Grams beside the diagonal contractions or after the update, at the edges of
their tiles and of the rule, and updates over one and many slices of partial sums."""
import pytest
import torch

import paper_1909_07570_amd as nnc

pytestmark = pytest.mark.gpu
EPS = 1e-12
SWEEPS = 3


def _unfold(x, n):
    return x.movedim(n, 0).reshape(x.shape[n], -1)


def _cp64(x, b):
    for _ in range(SWEEPS):
        for n in range(x.dim()):
            kr = None
            h = torch.ones(b[0].shape[1], b[0].shape[1], dtype=torch.float64)
            for k in range(x.dim()):
                if k != n:
                    kr = b[k] if kr is None else (kr[:, None, :] * b[k][None, :, :]).reshape(-1, b[k].shape[1])
                    h = h * (b[k].T @ b[k])
            b[n] = b[n] * (_unfold(x, n) @ kr) / (b[n] @ h).clamp_min(EPS)
    return b


@pytest.mark.parametrize(
    "dims,rank",
    [
        ((24, 7, 33), 1),  # below rank 4: Grams after the update
        ((24, 7, 33), 3),
        ((24, 7, 33), 4),
        ((24, 7, 33), 16),  # a full tile of ranks
        ((24, 7, 33), 17),  # two tiles
        ((19, 31, 6), 32),
        ((1024, 5, 6), 10),  # longest factor beside a contraction, and the next
        ((1025, 5, 6), 10),
        ((6, 1030, 4), 5),
        ((70, 130, 65), 10),  # several slices
        ((3, 5, 7, 9), 6),
        ((9, 300), 8),
    ],
)
def test_sweeps(dims, rank):
    gen = torch.Generator().manual_seed(sum(dims) + rank)
    x = torch.rand(*dims, generator=gen) + 1e-2
    b = [torch.rand(n, rank, generator=gen) + 1e-2 for n in dims]
    got = [t.cuda() for t in b]
    nnc.nncpx_fit(x.cuda(), rank, SWEEPS, got)
    want = _cp64(x.double(), [t.double() for t in b])
    # chains over a streamed mode, the other modes (at most their lengths together) and the ranks; a sweep
    # passes on what the ones before were off by, at most doubled
    tol = 2.0 ** -24 * (2 * sum(dims) + 2 * rank + 64) * (2 ** SWEEPS - 1)
    for g, w in zip(got, want):
        assert (g.double().cpu() - w).norm() <= tol * w.norm()
