"""Short contracted indices in rows that are no whole 16-byte chunks: the general kernel takes them, the
matrix-core ones the longer, and FP32 results are the same bits on both sides (products added in the
order of the contracted index); BF16 within N * 2^-24 of FP64."""
import zlib

import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu

# shape, mode, rank, whether the general kernel takes FP32 and BF16 X
CASES = [((20000, 20, 5), 1, 5, True, True), ((3000, 2, 9), 1, 9, True, True), ((9001, 1, 13), 1, 1, True, True),
         ((301, 187, 5, 5), 2, 4, True, True), ((30000, 9), 1, 3, True, True), ((2000, 301, 9), 1, 11, False, False),
         ((301, 250, 9), 1, 20, False, False), ((40000, 33), 1, 3, False, False), ((120, 9), 1, 3, False, False),
         ((500, 64, 130), 1, 20, False, False)]


@pytest.mark.parametrize("shape,mode,R,f32,bf16", CASES)
def test_either_side_of_the_line(shape, mode, R, f32, bf16):
    nnc = need_gpu()
    rng = np.random.default_rng(zlib.crc32(repr((shape, mode, R)).encode()))
    A = rng.random((shape[mode], R)).astype(np.float32)
    x = rng.random(shape).astype(np.float32)
    for dt, general in ((torch.float32, f32), (torch.bfloat16, bf16)):
        X64 = x.astype(np.float64) if dt == torch.float32 else synth.round_bf16(x.astype(np.float64))
        X = torch.from_numpy(X64).to("cuda").to(dt)
        print("case", shape, mode, R, dt, flush=True)
        got = nnc.nnc_ttm(X, mode, torch.from_numpy(A).to("cuda")).cpu().numpy()
        assert (nnc.last_ttm_kernel() == "ttm_generic") == general, nnc.last_ttm_kernel()
        y = np.moveaxis(X64, mode, -1).astype(np.float64)
        g = np.moveaxis(got, mode, -1)
        if dt == torch.float32:  # a chain of fused multiply-adds: exact products, one rounding a step
            want = np.zeros(y.shape[:-1] + (R,), np.float32)
            for n in range(shape[mode]):
                want = (want.astype(np.float64) + y[..., n:n + 1] * A[n].astype(np.float64)).astype(np.float32)
            # (a double sum rounded to float can differ from the fused step by a double rounding)
            assert (np.abs(g - want) <= 2.0 ** -23 * want).all() and (g != want).mean() <= 1e-3
        ref = np.stack([(y * A[:, r].astype(np.float64)).sum(axis=-1) for r in range(R)], axis=-1)
        assert (np.abs(g - ref) <= max(shape[mode], 16) * 2.0 ** -24 * ref).all()
