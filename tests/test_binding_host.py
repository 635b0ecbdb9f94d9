"""The binding's per-call look-ups and the layer's choice of the path without
autograd functions (no GPU needed)."""
import pytest
import torch
from torch.autograd import forward_ad

from paper_2307_02486_amd import DilatedAttnError, ops, plan
from paper_2307_02486_amd.layer import _plain


@pytest.mark.parametrize("patterns", [[(64, 1), (128, 2)], ((64, 1), (128, 2)), [[64, 1], [128, 2]],
                                      [(64.0, 1), (128, 2.0)]], ids=str)
def test_prepared_takes_every_form_of_patterns(patterns):
    want = max(256, plan(1, 256, 2, 32, [(64, 1), (128, 2)])["workspace_bytes"])
    for given in (patterns, iter(patterns)):
        got, arr, n = ops._prepared("dilated_attn_plan", (1, 256, 2, 32), given, 1, 1, 0.0)
        assert got == want and n == 2
        assert [(arr[i].w, arr[i].r) for i in range(n)] == [(64, 1), (128, 2)]


def test_prepared_refuses_what_the_plan_refuses():
    for bad in ([(4, 8)], [], [(0, 1)], [(8, 1)] * 17):
        for _ in range(2):  # an error is not remembered as a result
            with pytest.raises(DilatedAttnError):
                ops._prepared("dilated_attn_plan", (1, 256, 2, 32), bad, 1, 1, 0.0)


def test_workspace_lookup_raises_each_time():
    for _ in range(2):
        with pytest.raises(DilatedAttnError):
            ops._workspace_bytes("dilated_attn_wgrad_workspace", 64, 100, 128)
    assert ops._workspace_bytes("dilated_attn_layernorm_bwd_workspace", 0, 8) >= 0


def test_plain_only_without_recording_or_transforms():
    assert not _plain()
    with torch.no_grad():
        assert _plain()
        with forward_ad.dual_level():
            assert not _plain()
        seen = []
        torch.func.vmap(lambda x: seen.append(_plain()) or x)(torch.zeros(2))
        assert seen == [False]
    with torch.inference_mode():
        assert _plain()
