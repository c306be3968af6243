"""The matrix-core passes on X whose rows (or whose own first element, or the output's) do not
start at 16-byte boundaries, against FP64 products of the same inputs.

All terms are nonnegative, so FP32 accumulation of N of them is off by at most N * 2^-24
relative to each entry (the factor is applied exactly: in FP32, or as three bf16 parts that
sum to it), which is the tolerance.
"""
import zlib

import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu

# (shape, mode, R): rows of one chunk and one more element; just under and over the pieces of
# 8, 16 and 32 chunks; several tiles per wave; a contracted index of several chunks; columns
# just over one tile of 64 or 128, and fewer than one loader chunk's worth past it
CASES = [((70, 9), 1, 3), ((33, 11), 1, 16), ((1000, 63), 1, 5), ((513, 129), 1, 20), ((77, 187), 1, 7),
         ((40, 257), 1, 32), ((9001, 131), 1, 20), ((50, 2051), 1, 32), ((19, 4099), 1, 17),
         ((30, 9), 0, 4), ((31, 67), 0, 16), ((250, 129), 0, 20), ((64, 3, 255), 0, 32), ((5, 37, 131), 1, 11),
         ((1301, 133), 0, 20), ((2050, 71), 0, 32), ((300, 40, 187), 0, 11)]


@pytest.mark.parametrize("shape,mode,R", CASES)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_ragged_rows(shape, mode, R, dt, shift):
    nnc = need_gpu()
    rng = np.random.default_rng(zlib.crc32(repr((shape, mode, R, dt, shift)).encode()))
    X64 = synth.round_bf16(rng.random(shape)) if dt == "bf16" else rng.random(shape).astype(np.float32).astype(np.float64)
    n = X64.size
    buf = torch.zeros(n + 8, dtype=torch.bfloat16 if dt == "bf16" else torch.float32, device="cuda")
    buf[shift:shift + n] = torch.from_numpy(X64.ravel()).to("cuda").to(buf.dtype)
    X = buf[shift:shift + n].view(shape)
    A = rng.random((shape[mode], R)).astype(np.float32)
    osh = list(shape)
    osh[mode] = R
    m = int(np.prod(osh))
    obuf = torch.full((m + 16,), -7.0, device="cuda")
    out = obuf[shift:shift + m].view(osh)
    print("case", shape, mode, R, dt, shift, flush=True)
    nnc.nnc_ttm(X, mode, torch.from_numpy(A).to("cuda"), out=out)
    assert nnc.last_ttm_kernel() != "ttm_generic"
    ref = np.moveaxis(np.tensordot(X64, A.astype(np.float64), axes=(mode, 0)), -1, mode)
    got = out.double().cpu().numpy()
    err = np.abs(got - ref) / ref
    assert err.max() <= max(shape[mode], 16) * 2.0 ** -24, err.max()
    guard = obuf.cpu().numpy()
    assert (guard[:shift] == -7.0).all() and (guard[shift + m:] == -7.0).all()


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_ragged_rows_keep_infinities_to_their_rows(dt):
    """A row of X that holds an infinity leaves every other output row finite and exact."""
    nnc = need_gpu()
    rng = np.random.default_rng(5)
    X64 = synth.round_bf16(rng.random((200, 77)))
    A = rng.random((77, 5)).astype(np.float32)
    X = torch.from_numpy(X64).to("cuda").to(torch.bfloat16 if dt == "bf16" else torch.float32)
    ref = nnc.nnc_ttm(X, 1, torch.from_numpy(A).to("cuda"))
    X[101, :] = float("inf")
    X[13, 76] = float("inf")
    X[14, 0] = float("nan")
    out = nnc.nnc_ttm(X, 1, torch.from_numpy(A).to("cuda"))
    bad = ~torch.isfinite(out).all(dim=1)
    assert bad.nonzero().flatten().tolist() == [13, 14, 101]
    assert torch.equal(out[~bad], ref[~bad])
