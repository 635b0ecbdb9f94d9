"""Launches of 2^24 workgroups of 256 threads and more: in one grid dimension
they would be 2^32 work-items, past what it holds (and a launch beyond wraps
without an error).  One-row segments: every row attends to itself alone, so
out = v, lse = q.k / sqrt(D), dv = dout and dq = dk = 0."""
import pytest
import torch

import workloads
from tests.gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu
SHAPE = (1, (1 << 22) + 5, 4, 32)  # 2^24 + 20 items


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()
    yield
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=str)
def test_forward(dtype):
    """Float32: out is (p v) (1 / p) times the mix's weight of one, a few
    roundings of 2^-24 (2^-21 covers eight); lse within the rounding of 32
    products (2e-5).  bf16: out is v up to the fp16 the rows are kept in
    (2^-11 relative, plus 1e-6 for elements far below the row's largest)."""
    from paper_2307_02486_amd import dilated_attn
    note(f"[large launch] forward {dtype}")
    q, k, v = (workloads.make_random(SHAPE, dtype, 1.0, 79, "cuda", t) for t in range(3))
    out = torch.full_like(v, float("nan"))
    out, lse = dilated_attn(q, k, v, [(1, 1)], True, out=out)
    torch.cuda.synchronize()
    rel, floor = (2.0 ** -21, 0.0) if dtype == torch.float32 else (2.0 ** -11, 1e-6)
    assert bool(((out.float() - v.float()).abs() <= rel * v.float().abs() + floor).all())
    want = (q.float() * k.float()).sum(-1).mul_(SHAPE[3] ** -0.5).permute(0, 2, 1)
    assert float((lse - want).abs().max()) <= 2e-5


def test_backward():
    """P = 1 to float32's precision and bf16's exactly, so dv is dout as kept in
    fp16; dS = dP - delta differs from zero by the rounding of two sums of 32
    products (2e-5 covers it), times |k| or |q| <= 6, a scale of 0.18 and 32 terms."""
    from paper_2307_02486_amd import dilated_attn, dilated_attn_bwd
    note("[large launch] backward")
    q, k, v, dout = (workloads.make_random(SHAPE, torch.bfloat16, 1.0, 80, "cuda", t) for t in range(4))
    out, lse = dilated_attn(q, k, v, [(1, 1)], True)
    dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(3))
    dilated_attn_bwd(q, k, v, out, lse, dout, [(1, 1)], True, dq=dq, dk=dk, dv=dv)
    torch.cuda.synchronize()
    assert bool(((dv.float() - dout.float()).abs() <= 2.0 ** -8 * dout.float().abs() + 1e-6).all())
    assert float(dq.abs().max()) <= 1e-4 and float(dk.abs().max()) <= 1e-4


def test_layernorm_rows():
    """The largest row count, 2^26: the last rows and the first."""
    from paper_2307_02486_amd import layer_norm
    note("[large launch] layer norm")
    x = workloads.make_random((1 << 26, 8), torch.bfloat16, 1.0, 81, "cuda", 0)
    g = torch.ones(8, dtype=torch.bfloat16, device="cuda")
    y, mean, rstd = layer_norm(x, g, torch.zeros_like(g))
    torch.cuda.synchronize()
    for part in (slice(0, 64), slice((1 << 26) - 64, 1 << 26)):
        ref = torch.nn.functional.layer_norm(x[part].float(), (8,))
        assert float((y[part].float() - ref).abs().max()) <= 2.0 ** -8 * 3.0  # |y| < 3, one bf16 rounding
        assert float((mean[part] - x[part].float().mean(1)).abs().max()) <= 1e-5
