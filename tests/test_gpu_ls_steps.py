"""The least-squares steps of the real Tucker fit at the edges of their rank bounds and chunks,
continued from factors near the solution (well-conditioned systems), against the FP64 oracle.

With condition numbers near 1 the FP64 R x R algebra adds nothing visible; the FP32 contractions
(at most prod(dims) products, in trees and chains of a few hundred) leave each sweep's model off by
a few 2^-24 sqrt(chain length): 3 sweeps * d steps * 2^-24 * sqrt(1024) < 2e-5."""
import zlib

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import dev, host, need_gpu, rel_fro

pytestmark = pytest.mark.gpu

# ranks on each side of the kernels' multiples of four; fewer rows than one tile, a partial tile,
# rows over one and two chunks of 256; 2 to 4 modes; a core past the slice kernels' packing
CASES = [((9, 10, 11), (1, 1, 1)), ((9, 10, 11), (2, 2, 3)), ((40, 300, 17), (8, 9, 7)), ((33, 40, 520), (12, 13, 5)),
         ((30, 36, 44), (16, 17, 20)), ((48, 50, 52), (21, 24, 25)), ((64, 66, 68), (28, 29, 32)),
         ((300, 60), (20, 20)), ((12, 14, 10, 9), (3, 5, 4, 8))]


@pytest.mark.parametrize("dims,ranks", CASES)
def test_continued_fit_matches_oracle(dims, ranks):
    nnc = need_gpu()
    rng = np.random.default_rng(zlib.crc32(repr((dims, ranks)).encode()))
    A = [np.linalg.qr(rng.standard_normal((n, r)))[0] for n, r in zip(dims, ranks)]
    G = rng.uniform(-1, 1, ranks)
    X = (oracle.tucker_full(G, A) + 1e-4 * rng.uniform(-1, 1, dims)).astype(np.float32)
    G0 = (G + 0.02 * rng.uniform(-1, 1, ranks)).astype(np.float32)
    A0 = [(a + 0.02 / np.sqrt(a.shape[0]) * rng.uniform(-1, 1, a.shape)).astype(np.float32) for a in A]
    print("case", dims, ranks, flush=True)
    Gd, Ad = dev(G0), [dev(a) for a in A0]
    rep = nnc.tucker_ls_fit(dev(X), ranks, 3, Gd, Ad)
    Go, Ao, _ = oracle.tucker_ls(X.astype(np.float64), G0, A0, 3)
    assert rel_fro(oracle.tucker_full(host(Gd), [host(a) for a in Ad]), oracle.tucker_full(Go, Ao)) <= 2e-5
    for a, ao in zip(Ad, Ao):
        assert rel_fro(host(a), ao) <= 2e-4
        assert np.abs(host(a).T @ host(a) - np.eye(ao.shape[1])).max() <= 1e-5
    assert abs(rep.rel_residual - oracle.tucker_rel_residual(X.astype(np.float64), Go, Ao)) <= 2e-5


def test_systems_that_are_not_definite_are_reported():
    """A zero core makes every K_n singular: the call reports it, whatever the rank's bound."""
    nnc = need_gpu()
    for r in (2, 9, 20, 32):
        X = dev(np.random.default_rng(r).standard_normal((36, 34, 40)).astype(np.float32))
        G = dev(np.zeros((r, r, r), np.float32))
        A = [dev(np.random.default_rng(r + k).standard_normal((n, r)).astype(np.float32)) for k, n in enumerate((36, 34, 40))]
        with pytest.raises(nnc.NncError) as e:
            nnc.tucker_ls_fit(X, (r, r, r), 2, G, A)
        assert e.value.status == nnc.NNC_ENUMERIC
