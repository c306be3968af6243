"""The kernel names of ragged contractions, in one launch and in several."""
import pytest
import torch

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,mode,R,what", [((77, 187), 1, 7, "ragged"), ((50, 2051), 1, 32, "ragged, chunked"),
                                               ((19, 4099), 1, 17, "ragged, chunked"), ((31, 67), 0, 16, "ragged"),
                                               ((1301, 133), 0, 20, "ragged, chunked"), ((64, 3, 255), 0, 32, "ragged")])
@pytest.mark.parametrize("dt,name", [(torch.float32, "f32"), (torch.bfloat16, "bf16")])
def test_names(shape, mode, R, what, dt, name):
    nnc = need_gpu()
    nnc.nnc_ttm(torch.ones(shape, device="cuda").to(dt), mode, torch.ones(shape[mode], R, device="cuda"))
    kind = "ttm_mid_" if mode < len(shape) - 1 else "ttm_last_lds_"
    assert nnc.last_ttm_kernel() == "%s%s (%s)" % (kind, name, what)
