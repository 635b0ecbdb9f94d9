"""The float32 attention kernel at the edges of its tiles: 64-query items of two
32-query blocks, keys dealt to two waves in 32-key blocks and merged at the end.

Bar: float32 throughout.  With |scores| <= 8 and |v| <= 5 a row's output is a
convex combination of v; the error is that of the scores (D products, about
2^-24 sqrt(D) |q||k| / sqrt(D) <= 4e-6), of the exponentials (2^-22 relative)
and of the final sums: below 2e-5.  lse inherits the scores' error: 2e-5.
"""
import pytest
import torch

import workloads
from tests.gpu_util import compare_full, note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


CASES = [(n, D, causal) for n in (31, 33, 64, 65, 97, 128, 161) for D in (32, 64, 128) for causal in (True, False)]


@pytest.mark.parametrize("n,D,causal", CASES, ids=str)
def test_tile_edges(n, D, causal):
    note(f"[f32] N={n} D={D} causal={causal}")
    q, k, v = (workloads.make_random((2, n, 3, D), torch.float32, 1.0, 50 + n, "cuda", t) for t in range(3))
    compare_full(q, k, v, [(n, 1), (n // 2 + 1, 2)], causal, "f32", tag=f"N{n} D{D}", tol=(2e-5, 2e-5))


@pytest.mark.parametrize("causal", [True, False])
def test_long_rows_with_growing_scores(causal):
    """Key blocks whose maxima keep rising: both halves rescale, and the merge
    weights differ widely."""
    N, D = 700, 64
    note(f"[f32] growing scores causal={causal}")
    q, k, v = (workloads.make_random((1, N, 2, D), torch.float32, 1.0, 77, "cuda", t) for t in range(3))
    k = k * torch.linspace(0.1, 6.0, N, device="cuda")[None, :, None, None]
    # scores reach about 40 here: their float32 error scales with them
    compare_full(q, k.contiguous(), v, [(N, 1), (N, 3)], causal, "f32", tag="growing", tol=(1e-4, 1e-4))


def test_wide_row_stride():
    """r * H * D so large that a 64-key tile spans 2 GiB: 64-bit addresses."""
    note("[f32] wide stride")
    q, k, v = (workloads.make_random((1, 96, 1024, 128), torch.float32, 1.0, 78, "cuda", t) for t in range(3))
    compare_full(q, k, v, [(96, 32)], True, "f32", tag="wide", tol=(2e-5, 2e-5))
