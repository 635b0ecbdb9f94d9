"""The layer without gradients calls the kernels directly and rotates q and k
in place: the same bits as through the autograd functions."""
import pytest
import torch

import workloads
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=str)
@pytest.mark.parametrize("use_xpos", [True, False])
@pytest.mark.parametrize("strided", [False, True])
def test_no_grad_forward_is_the_same(dtype, use_xpos, strided):
    from paper_2307_02486_amd.layer import LongNetAttention
    note(f"[plain] {dtype} xpos={use_xpos} strided={strided}")
    torch.manual_seed(1)
    layer = LongNetAttention(128, 2, [(64, 1), (150, 3)], use_xpos=use_xpos, device="cuda", dtype=dtype)
    x = workloads.make_random((2, 150, 128), dtype, 1.0, 61, "cuda", 0)
    if strided:
        x = x.transpose(0, 1).contiguous().transpose(0, 1)
    with torch.enable_grad():
        want = layer(x).detach()
    before = x.clone()
    with torch.no_grad():
        got = layer(x)
    assert torch.equal(got, want) and torch.equal(x, before)
    with torch.inference_mode():
        assert torch.equal(layer(x), want)
