"""Infinities and NaN in X whose rows do not start at 16-byte boundaries: every output entry is the
infinity, the NaN or the finite sum that its own products give (zero times an infinity among them),
whatever the kernels multiply beside them.  Finite entries within N * 2^-24 of FP64, as for any X."""
import zlib

import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu

# the last mode and earlier ones, one and two rank tiles, one chunk of the contracted index and several
CASES = [((200, 77), 1, 5), ((33, 11), 1, 16), ((40, 257), 1, 20), ((50, 2051), 1, 32), ((19, 4099), 1, 17),
         ((31, 67), 0, 16), ((40, 3, 255), 0, 32), ((5, 37, 131), 1, 11), ((1301, 133), 0, 20)]


@pytest.mark.parametrize("shape,mode,R", CASES)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("factor", ["random", "eighths"])  # eighths: values that bf16 holds, some zero
def test_infinities_are_what_their_sums_give(shape, mode, R, dt, factor):
    nnc = need_gpu()
    rng = np.random.default_rng(zlib.crc32(repr((shape, mode, R, dt, factor)).encode()))
    X64 = synth.round_bf16(rng.random(shape)) if dt == "bf16" else rng.random(shape).astype(np.float32).astype(np.float64)
    A = rng.random((shape[mode], R)).astype(np.float32)
    if factor == "eighths":
        A = np.maximum(np.round(8 * A) - 1, 0).astype(np.float32) / 8
    x = np.moveaxis(X64, mode, -1)  # rows of the contracted index
    flat = [np.unravel_index(i, x.shape[:-1]) for i in rng.permutation(int(np.prod(x.shape[:-1])))[:9]]
    n = shape[mode]
    x[flat[0] + (0,)] = np.inf
    x[flat[1] + (n - 1,)] = np.inf
    x[flat[2] + (n // 2,)] = -np.inf
    x[flat[3] + (0,)], x[flat[3] + (n - 1,)] = np.inf, -np.inf
    x[flat[4] + (n // 3,)] = np.nan
    x[flat[5]] = np.inf
    X = torch.from_numpy(X64).to("cuda").to(torch.bfloat16 if dt == "bf16" else torch.float32)
    print("case", shape, mode, R, dt, factor, flush=True)
    got = nnc.nnc_ttm(X, mode, torch.from_numpy(A).to("cuda"))
    assert nnc.last_ttm_kernel() != "ttm_generic"
    got = np.moveaxis(got.double().cpu().numpy(), mode, -1)
    with np.errstate(invalid="ignore"):
        ref = np.stack([(x * A[:, r].astype(np.float64)).sum(axis=-1) for r in range(R)], axis=-1)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    assert np.isinf(ref).any() and np.isnan(ref).any()
    ok = np.isfinite(ref)
    assert (np.abs(got[ok] - ref[ok]) <= max(n, 16) * 2.0 ** -24 * ref[ok]).all()
