"""The quotient of the NMF's multiplicative updates, x * num / max(den, eps), is the float of the double
division for every value: independent numerators and denominators, and quotients that lie exactly
between two floats.  W's update of one sweep, whose FP32 products the host repeats exactly."""
import numpy as np
import pytest
import torch

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu
ROWS = 512


def _w_after(nnc, A, W, H, eps):
    w = torch.from_numpy(W.copy()).to("cuda")
    nnc.nmf_fit(torch.from_numpy(A).to("cuda"), W.shape[1], 1, w, torch.from_numpy(H).to("cuda"), eps=eps, residual=False)
    return w.cpu().numpy()


@pytest.mark.parametrize("span", [3, 60])
def test_independent_numerators_and_denominators(span):
    nnc = need_gpu()
    rng = np.random.default_rng(11)
    wrong = 0
    for i in range(256):
        h = np.float32(np.exp(rng.uniform(-2, 2)))
        x = np.exp(rng.uniform(-span, span, ROWS)).astype(np.float32)
        a = np.exp(rng.uniform(-20, 20, ROWS)).astype(np.float32)
        num, den = a * h, x * np.float32(h * h)  # one rounding each, as there
        want = (x.astype(np.float64) * num.astype(np.float64) / np.maximum(den.astype(np.float64), 1e-37)).astype(np.float32)
        got = _w_after(nnc, a[:, None], x[:, None], np.full((1, 1), h, np.float32), 1e-37)[:, 0]
        wrong += int((got != want).sum())
    assert wrong == 0


@pytest.mark.parametrize("m,col", [(2, 0), (18, 16)])  # entries of the matrix cores, and of the tail of ranks
def test_quotients_halfway_between_floats(m, col):
    """Columns col, col + 1 of W are [3 D, D], the others zero, and H = 1/2: num = a / 2 and
    den = D exactly, so the first becomes 3 a / 2, which for odd a between 2^24 / 3 and 2^25 / 3 is
    halfway between two floats."""
    nnc = need_gpu()
    rng = np.random.default_rng(12)
    wrong = 0
    for i in range(64):
        D = (2 * rng.integers(1, 1 << 21, ROWS) + 1).astype(np.float32)
        a = (2 * rng.integers(2796203, 5592405, ROWS) + 1).astype(np.float32)
        W, H = np.zeros((ROWS, m), np.float32), np.full((m, 1), 0.5, np.float32)
        W[:, col], W[:, col + 1] = 3 * D, D
        want = (1.5 * a.astype(np.float64)).astype(np.float32)  # to even
        assert np.all(want != 1.5 * a.astype(np.float64))
        wrong += int((_w_after(nnc, a[:, None], W, H, 1e-12)[:, col] != want).sum())
    assert wrong == 0


def test_values_that_take_the_division():
    nnc = need_gpu()

    def one(x, a, h, eps):
        A, W, H = (np.full((1, 1), v, np.float32) for v in (a, x, h))
        return _w_after(nnc, A, W, H, eps)[0, 0]

    inf = np.float32(np.inf)
    assert one(1.0, 1.0, 1.0, 1e39) == np.float32(1e-39)  # an eps above every float clips every denominator
    assert one(3e38, 1.0, 2.0, 1e39) == 0.0  # over an infinite denominator
    assert one(2.0, inf, 1.0, 1e-12) == inf
    assert np.isnan(one(inf, 1.0, 1.0, 1e-12))  # inf / inf
    assert np.isnan(one(1.0, np.float32(np.nan), 1.0, 1e-12))
