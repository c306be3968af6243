"""nnCP of the core on the matrix cores at the edges of its tiles, groups and variants, against
the FP64 oracle from the same starts.

After three sweeps from nonnegative data, every value is a product of FP32 sums of at most
prod(dims) nonnegative terms, each off by at most 2^-24 times its number of steps; with the
pairwise shortness of the real chains, (number of modes) * 3 sweeps * sqrt(prod(dims)) * 2^-24 * 4
bounds the relative Frobenius error with room."""
import zlib

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import dev, host, need_gpu, rel_fro

pytestmark = pytest.mark.gpu

# one row and one column; just under and over tiles of 16 and steps of 4; ranks over 16; every
# order with its groups; fragments in registers (16, 32 a lane) and streamed; modes at the limit
# of 64 and over it (the general kernel)
CASES = [((1, 1), 1), ((8, 8, 8), 7), ((11, 47, 1), 3), ((4, 2, 64), 20), ((2, 3), 2), ((17, 5), 7), ((64, 64), 32), ((65, 9), 4), ((3, 4, 5), 5), ((16, 4, 4), 16),
         ((17, 15, 5), 17), ((20, 20, 20), 10), ((24, 24, 24), 16), ((33, 2, 31), 32), ((5, 4, 3, 2), 3),
         ((16, 16, 16, 16), 8), ((9, 7, 11, 5), 16), ((8, 8, 8, 8, 8), 16), ((7, 2, 3, 5, 4), 9),
         ((3, 4, 2, 5, 3, 4), 6), ((2, 2, 2, 2, 2, 2, 2), 3)]


@pytest.mark.parametrize("dims,r", CASES)
def test_few_sweeps_match_oracle(dims, r):
    nnc = need_gpu()
    rng = np.random.default_rng(zlib.crc32(repr((dims, r)).encode()))
    T = (oracle.cp_full([rng.random((n, min(r, 4))) for n in dims]) + 0.1 * rng.random(dims)).astype(np.float32)
    B0 = synth.init_cp_factors(170, dims, r)
    Bo, clips, _ = oracle.nncp(T.astype(np.float64), B0, 3)
    B = [dev(b) for b in B0]
    print("case", dims, r, flush=True)
    rep = nnc.nncp_fit(dev(T), r, 3, B, report=True)
    assert rep.eps_clips == clips
    tol = len(dims) * 3 * np.sqrt(np.prod(dims)) * 2.0 ** -24 * 4 + 1e-6
    for b, bo in zip(B, Bo):
        assert rel_fro(host(b), bo) <= tol, (rel_fro(host(b), bo), tol)
    assert abs(rep.rel_residual - oracle.cp_rel_residual(T.astype(np.float64), Bo)) <= tol
    B = [dev(b) for b in B0]
    assert abs(nnc.nncp_fit(dev(T), r, 0, B) - oracle.cp_rel_residual(T.astype(np.float64), B0)) <= tol
    assert all(np.array_equal(host(b), b0) for b, b0 in zip(B, B0))


@pytest.mark.parametrize("threads", [64, 192, 256, 320, 512, 1024])
@pytest.mark.parametrize("dims", [(20, 18, 7), (6, 5, 4, 7), (5, 4, 6, 3, 5)])
def test_thread_counts_and_uneven_ranks(dims, threads):
    nnc = need_gpu()
    rng = np.random.default_rng(zlib.crc32(repr((dims, threads)).encode()))
    T = (oracle.cp_full([rng.random((n, 4)) for n in dims]) + 0.1 * rng.random(dims)).astype(np.float32)
    ranks = [1, 4, 19, 9]
    inits = [synth.init_cp_factors(171, dims, r, restart=j) for j, r in enumerate(ranks)]
    facs = [[dev(b) for b in B0] for B0 in inits]
    print("case", dims, threads, flush=True)
    res = nnc.nncp_fit_batched(dev(T), ranks, 3, facs, threads_per_fit=threads)
    tol = len(dims) * 3 * np.sqrt(np.prod(dims)) * 2.0 ** -24 * 4 + 1e-6
    for j in range(len(ranks)):
        Bo, _, _ = oracle.nncp(T.astype(np.float64), inits[j], 3)
        assert abs(res[j] - oracle.cp_rel_residual(T.astype(np.float64), Bo)) <= tol
        for b, bo in zip(facs[j], Bo):
            assert rel_fro(host(b), bo) <= tol


def test_tensor_placement_changes_no_result(tmp_path, monkeypatch):
    """A choice of the tensor in global memory, from a tuner file, changes no result."""
    nnc = need_gpu()
    import torch
    p = torch.cuda.get_device_properties(0)
    tag = "%s/%dcu" % (p.gcnArchName.split(":")[0], p.multi_processor_count)
    rng = np.random.default_rng(172)
    dims, ranks = (8, 7, 6, 9), [3, 12]
    T = dev(rng.random(dims).astype(np.float32))
    got = []
    for tg in (0, 1):
        path = tmp_path / ("t%d.json" % tg)
        path.write_text('{"key": "%s|8x7x6x9|3,12", "threads": 512, "t_global": %d, "lpt": 0, "ms": 1.0}\n' % (tag, tg))
        monkeypatch.setenv("NNC_TUNE_CACHE", str(path))
        facs = [[dev(b) for b in synth.init_cp_factors(172, dims, r, restart=j)] for j, r in enumerate(ranks)]
        res = nnc.nncp_fit_batched(T, ranks, 7, facs)
        assert nnc.last_tune()["t_global"] == tg
        got.append((res, [host(b) for f in facs for b in f]))
    assert got[0][0] == got[1][0]
    assert all(np.array_equal(x, y) for x, y in zip(got[0][1], got[1][1]))
