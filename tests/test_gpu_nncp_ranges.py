"""nnCP of cores whose left modes are short and right modes long on the matrix cores: V's few tiles are
split into ranges of the contracted index while the tensor is read from the L2, at every thread count,
against the FP64 oracle from the same starts.  The tolerance is that of the kernel's other few-sweep
tests: FP32 sums of nonnegative terms, (number of modes) * 3 sweeps * sqrt(prod(dims)) * 2^-24 * 4."""
import zlib

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import dev, host, need_gpu, rel_fro

pytestmark = pytest.mark.gpu


def _case(dims, ranks):
    rng = np.random.default_rng(zlib.crc32(repr((dims, ranks)).encode()))
    T = (oracle.cp_full([rng.random((n, 4)) for n in dims]) + 0.1 * rng.random(dims)).astype(np.float32)
    inits = [synth.init_cp_factors(173, dims, r, restart=j) for j, r in enumerate(ranks)]
    tol = len(dims) * 3 * np.sqrt(np.prod(dims)) * 2.0 ** -24 * 4 + 1e-6
    return T, inits, tol


# ranges of 8, 4 and 2, a single tile and more, the last range shorter, one row past a tile
@pytest.mark.parametrize("dims,r", [((4, 4, 16, 16), 8), ((5, 5, 12, 12), 10), ((8, 8, 11, 12), 6), ((4, 8, 12, 16), 17),
                                    ((4, 16, 16, 16), 8), ((3, 4, 9, 9), 5), ((5, 6, 9, 9), 4), ((17, 1, 13, 11), 9),
                                    ((2, 2, 64, 64), 3), ((8, 4, 64, 32), 8), ((2, 3, 4, 12, 12), 9),
                                    ((3, 3, 4, 12, 12), 8)])
def test_streamed_ranges_match_oracle(dims, r):
    nnc = need_gpu()
    T, (B0,), tol = _case(dims, [r])
    Bo, clips, _ = oracle.nncp(T.astype(np.float64), B0, 3)
    B = [dev(b) for b in B0]
    print("case", dims, r, flush=True)
    rep = nnc.nncp_fit(dev(T), r, 3, B, report=True)
    assert rep.eps_clips == clips
    for b, bo in zip(B, Bo):
        assert rel_fro(host(b), bo) <= tol, (rel_fro(host(b), bo), tol)
    assert abs(rep.rel_residual - oracle.cp_rel_residual(T.astype(np.float64), Bo)) <= tol


@pytest.mark.parametrize("threads", [128, 192, 256, 512, 1024])
@pytest.mark.parametrize("dims", [(5, 6, 9, 9), (4, 4, 40), (1, 9, 57), (4, 5, 20, 20)])
def test_streamed_ranges_at_thread_counts(dims, threads):
    nnc = need_gpu()
    ranks = [3, 16, 7]
    T, inits, tol = _case(dims, ranks)
    facs = [[dev(b) for b in B0] for B0 in inits]
    print("case", dims, threads, flush=True)
    res = nnc.nncp_fit_batched(dev(T), ranks, 3, facs, threads_per_fit=threads)
    for j in range(len(ranks)):
        Bo, _, _ = oracle.nncp(T.astype(np.float64), inits[j], 3)
        assert abs(res[j] - oracle.cp_rel_residual(T.astype(np.float64), Bo)) <= tol
        for b, bo in zip(facs[j], Bo):
            assert rel_fro(host(b), bo) <= tol


@pytest.mark.parametrize("dims,r", [((33, 33, 33), 3), ((40, 40, 40), 8), ((21, 38, 61), 10), ((21, 38, 61), 11),
                                    ((9, 8, 8), 17), ((9, 8, 8), 23), ((2, 1, 51, 39), 8), ((7, 2, 53, 38), 3)])
def test_either_side_of_the_lines_matches_oracle(dims, r):
    """Shapes on both sides of the lines between this kernel and the one-contraction kernel."""
    nnc = need_gpu()
    T, (B0,), tol = _case(dims, [r])
    Bo, _, _ = oracle.nncp(T.astype(np.float64), B0, 3)
    B = [dev(b) for b in B0]
    print("case", dims, r, flush=True)
    res = nnc.nncp_fit(dev(T), r, 3, B)
    for b, bo in zip(B, Bo):
        assert rel_fro(host(b), bo) <= tol, (rel_fro(host(b), bo), tol)
    assert abs(res - oracle.cp_rel_residual(T.astype(np.float64), Bo)) <= tol
