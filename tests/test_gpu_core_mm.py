"""Small contractions by 16, 32 and 64 pairs a block, and core slices contracted on the matrix cores, at
the edges of their tiles, against FP64 sweeps of the same start."""
import numpy as np
import pytest
import torch

from oracle import nntucker
from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu
SWEEPS = 2


@pytest.mark.parametrize(
    "dims,ranks",
    [
        ((9, 8, 7), (1, 1, 1)),
        ((17, 40, 33), (4, 5, 3)),
        ((40, 33, 24), (8, 8, 8)),  # full rows of ranks
        ((40, 33, 50), (16, 17, 15)),  # one and two tiles of ranks
        ((36, 45, 64), (24, 20, 9)),
        ((34, 32, 48), (32, 32, 16)),
        ((510, 100, 34), (6, 5, 32)),  # 16320 pairs, four waves a block: tiles of 16
        ((513, 100, 34), (6, 5, 32)),  # 16416: tiles of 32
        ((200, 500, 34), (6, 5, 32)),  # 6400, sixteen waves: tiles of 32
        ((300, 500, 34), (6, 5, 32)),  # 9600: tiles of 64
        ((12, 10, 11, 9), (3, 4, 5, 6)),
        ((20, 18, 17, 19), (16, 15, 16, 13)),  # slices of several tiles a wave, one core row a block
        ((6, 7, 5, 6, 8), (2, 5, 3, 4, 3)),
    ],
)
def test_sweeps(dims, ranks):
    nnc = need_gpu()
    rng = np.random.default_rng(sum(dims) + sum(ranks))
    X = (rng.random(dims) + 1e-2).astype(np.float32)
    G = (rng.random(ranks) + 1e-2).astype(np.float32)
    A = [(rng.random((n, r)) + 1e-2).astype(np.float32) for n, r in zip(dims, ranks)]
    got_g, got_a = torch.from_numpy(G).cuda(), [torch.from_numpy(a).cuda() for a in A]
    nnc.nntucker_fit(torch.from_numpy(X).cuda(), list(ranks), SWEEPS, got_g, got_a)
    out = nntucker(X.astype(np.float64), G.astype(np.float64), [a.astype(np.float64) for a in A], SWEEPS)
    want_g, want_a = out[0], out[1]
    # All terms are nonnegative: a chain of n sums is off by at most n 2^-24.  An update has chains over the
    # modes, the ranks and the entries of a core slice (32 or more threads to one); a later update passes on
    # what those before it were off by, each sweep at most doubling it.
    slices = max(int(np.prod(ranks)) // r for r in ranks)
    tol = 2.0 ** -24 * (2 * sum(dims) + 4 * sum(ranks) + slices // 16) * (2 ** SWEEPS - 1)
    for g, w in zip([got_g] + got_a, [want_g] + list(want_a)):
        assert np.linalg.norm(g.double().cpu().numpy() - w) <= tol * np.linalg.norm(w)
