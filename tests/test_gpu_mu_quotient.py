"""The quotient of the NMF's multiplicative updates, x * num / max(den, eps) in double rounded to float,
against an exact division, through one sweep of the NMF of a 1 x 1 matrix at rank 1:
W <- W (A H) / (W H H), with FP32 products exactly as here, so the float must be the division's
except where the exact quotient lies within 2^-28 of a rounding boundary (about 2 of 2^27 values)."""
import numpy as np
import pytest
import torch

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def test_quotients_round_as_the_division_does():
    nnc = need_gpu()
    rng = np.random.default_rng(7)
    n = 1 << 20
    x = np.exp(rng.uniform(-60, 60, n)).astype(np.float32)
    a = np.exp(rng.uniform(-20, 20, n)).astype(np.float32)
    # rows of a rank-1 NMF with H = 1: num = a, den = w * 1 (one product each, exact)
    W = torch.from_numpy(x[:, None].copy()).to("cuda")
    A = torch.from_numpy(a[:, None].copy()).to("cuda")
    rows = 512
    wrong = 0
    for i in range(0, 1 << 16, rows):
        w, h = W[i:i + rows].clone().contiguous(), torch.ones(1, 1, device="cuda")
        nnc.nmf_fit(A[i:i + rows].contiguous(), 1, 1, w, h, eps=1e-37, residual=False)
        xs, an = x[i:i + rows].astype(np.float64), a[i:i + rows].astype(np.float64)
        want = (xs * an / np.maximum(xs, 1e-37)).astype(np.float32)
        got = w.cpu().numpy()[:, 0]
        wrong += int((got != want).sum())
        assert np.all(np.abs(got.astype(np.float64) - want) <= 1.2e-7 * want)
    assert wrong <= 1, wrong


def test_extreme_denominators():
    """A zero numerator over a clipped denominator is zero, a huge quotient infinite, and one over a
    large denominator what the division gives."""
    nnc = need_gpu()

    def one(x, a, eps):
        w, h = torch.full((1, 1), x, device="cuda"), torch.ones(1, 1, device="cuda")
        nnc.nmf_fit(torch.full((1, 1), a, device="cuda"), 1, 1, w, h, eps=eps, residual=False)
        return float(w.item())

    assert one(0.0, 1.0, 1e-310) == 0.0
    assert one(1.0, 0.0, 1e-12) == 0.0
    assert one(1e-30, 1e30, 1e-12) == np.float32(np.float64(np.float32(1e-30)) * np.float64(np.float32(1e30)) / 1e-12)
    assert one(3e38, 3e38, 1e-12) == np.float32(3e38)
    assert np.isnan(one(float("nan"), 1.0, 1e-12))
