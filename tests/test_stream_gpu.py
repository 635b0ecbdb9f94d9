"""The binding's raw stream is torch's current one, and calls follow it."""
import pytest
import torch

import workloads
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def test_raw_stream_is_the_current_one():
    from paper_2307_02486_amd import ops
    dev = torch.device("cuda", torch.cuda.current_device())
    note("[stream] raw stream")
    assert ops._raw_stream(dev) == torch.cuda.current_stream(dev).cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert ops._raw_stream(dev) == side.cuda_stream == torch.cuda.current_stream(dev).cuda_stream
    assert ops._raw_stream(dev) == torch.cuda.current_stream(dev).cuda_stream


def test_a_given_stream_gives_the_same_bits(monkeypatch):
    """Each entry point on a stream that is not the current one (its inputs made
    and waited for before), against the current one.  Every tensor it returns
    is recorded for that stream: the binding allocated it on the current one."""
    from paper_2307_02486_amd import ops
    from paper_2307_02486_amd import dilated_attn, dilated_attn_bwd, layer_norm, layer_norm_bwd, wgrad, xpos
    note("[stream] given stream")
    q, k, v, dout = (workloads.make_random((1, 300, 4, 64), torch.bfloat16, 1.0, 90, "cuda", t) for t in range(4))
    x, dy = (t.reshape(300, 256) for t in (q, dout))
    g = workloads.make_random((256,), torch.bfloat16, 1.0, 91, "cuda", 0)
    pats = [(128, 1), (300, 3)]

    def calls(stream):
        out, lse = dilated_attn(q, k, v, pats, stream=stream)
        yield out, lse
        yield dilated_attn_bwd(q, k, v, out, lse, dout, pats, stream=stream)
        yield (xpos(q, 1, stream=stream),)
        y, mean, rstd = layer_norm(x, g, g, stream=stream)
        yield y, mean, rstd
        yield layer_norm_bwd(dy, x, g, mean, rstd, stream=stream)
        yield wgrad(dy, x, bias_grad=True, stream=stream)

    want = [t for ts in calls(None) for t in ts]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    owned = []
    record = ops._stream_use

    def use(stream, tensors):
        owned.extend(t.data_ptr() for t in tensors)
        record(stream, tensors)

    monkeypatch.setattr(ops, "_stream_use", use)
    got = [t for ts in calls(side) for t in ts]
    torch.cuda.synchronize()
    assert {t.data_ptr() for t in got} <= set(owned)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
