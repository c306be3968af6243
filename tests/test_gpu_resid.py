"""Residual sums and model expansions at the edges of their tiles against FP64 products.

The model values are FP32 sums of R products of d FP32 values: off by at most (R + d) * 2^-23
of themselves for nonnegative terms.  ||X - Xhat||^2 of unrelated X and Xhat then moves by at
most 2 (R + d) 2^-23 (||Xhat|| / ||X - Xhat||) relative, the tolerance; ||X||^2 is an FP64 sum
of exact squares."""
import zlib

import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import bf16_dev, dev, need_gpu

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (3, 2), (17, 3), (5, 63), (16, 64), (33, 65), (15, 127), (70, 128), (4, 5, 129), (31, 187), (9, 513),
          (2, 3, 1100), (21, 22, 23), (6, 7, 8, 64), (3, 4, 5, 6, 7)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("R", [1, 4, 7, 20, 29, 32])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("model", ["cp", "tucker"])
def test_sums(shape, R, dt, model):
    nnc = need_gpu()
    if model == "tucker" and R ** len(shape) > 1 << 17:
        R = {3: 20, 4: 7, 5: 4}[len(shape)]
    rng = np.random.default_rng(zlib.crc32(repr((shape, R, dt, model)).encode()))
    X64 = synth.round_bf16(rng.random(shape)) if dt == "bf16" else rng.random(shape).astype(np.float32).astype(np.float64)
    X = bf16_dev(X64) if dt == "bf16" else dev(X64.astype(np.float32))
    d = len(shape)
    A = [rng.random((n, R)).astype(np.float32) for n in shape]
    G = None
    if model == "cp":
        hat = np.einsum(*[v for k in range(d) for v in (A[k].astype(np.float64), [k, 20])], list(range(d)))
    else:
        G = rng.random((R,) * d).astype(np.float32)
        hat = G.astype(np.float64)
        for k in range(d):
            hat = np.moveaxis(np.tensordot(hat, A[k].astype(np.float64), axes=(k, 1)), -1, k)
    print("case", shape, R, dt, model, flush=True)
    e, n = nnc.reconstruct_sq_sums(X, [dev(a) for a in A], dev(G) if G is not None else None)
    e_ref, n_ref = float(((X64 - hat) ** 2).sum()), float((X64 ** 2).sum())
    terms = R * d if model == "tucker" else R
    tol = 2 * (terms + d) * 2.0 ** -23 * np.sqrt((hat ** 2).sum() / e_ref)
    assert abs(e - e_ref) <= tol * e_ref, (e, e_ref)
    assert abs(n - n_ref) <= 1e-12 * n_ref


def test_rows_past_a_nan_do_not_spread():
    """X with a NaN is reported, and a finite X of a ragged size is not."""
    nnc = need_gpu()
    A = [torch.rand(n, 5, device="cuda") for n in (9, 10, 67)]
    X = torch.rand(9, 10, 67, device="cuda")
    assert np.isfinite(nnc.reconstruct_residual(X, A))
    X[8, 9, 66] = float("nan")
    with pytest.raises(nnc.NncError):
        nnc.reconstruct_residual(X, A)
