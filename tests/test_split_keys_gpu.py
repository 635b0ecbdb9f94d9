"""The bf16 forward's two forms: 64-row items whose keys are split over two
waves (launches too small to fill the chip) and 128-row items, each against
the oracle where it can go wrong.  Bars: those of the bf16 parity tests
(2e-2 on out, 1e-2 on lse: bf16 probabilities and outputs of size about 1)."""
import pytest
import torch

import workloads
from tests.gpu_util import compare_full, note, require_gpu
from tests.test_parity_gpu import LOG2E, REGIME_SCALES, _integer_qkv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 65, 96, 97, 129, 193])
def test_split_tile_edges(n, D, causal):
    """Rows and keys at the edges of 32-query blocks, 32-key halves and 64-key
    tiles: halves that see no key, segments that end inside either half."""
    note(f"[split] N={n} D={D} causal={causal}")
    q, k, v = (workloads.make_random((1, n, 3, D), torch.bfloat16, 1.0, 300 + n, "cuda", t) for t in range(3))
    compare_full(q, k, v, [(n, 1), (max(2, n // 2 + 1), 2)], causal, "bf16", tag=f"N{n} D{D}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("regime,jump", [("rescale", 2.0), ("rerun", 8.0), ("overflow", 16.0)])
@pytest.mark.parametrize("H", [2, 80])
def test_growing_scores_in_both_forms(H, D, causal, regime, jump):
    """Scores that grow along the sequence with 2 heads (split keys) and with
    80 copies of them (640 items for one pattern alone: 128-row items)."""
    note(f"[split] {regime} H={H} D={D} causal={causal}")
    q, k, v = (x.repeat(1, 1, H // 2, 1) for x in _integer_qkv(1, 1000, 2, D, seed=31 + D, jump_at=300, jump=jump))
    compare_full(q, k, v, [(1000, 1), (500, 2)], causal, "bf16", scale=REGIME_SCALES["generic"] / LOG2E,
                 tag=f"{regime} H{H} D{D}", heads=[0, 1])


@pytest.mark.parametrize("H", [17, 136])
def test_wide_row_stride_in_both_forms(H):
    """64-bit addressing (key tiles spanning 2 GiB) in both forms."""
    note(f"[split] wide stride H={H}")
    r = -(-65536 // H)  # r * H * 128 columns * 2 bytes * 129 rows >= 2^31
    N = 5 * r
    q, k, v = (workloads.make_random((1, N, H, 128), torch.bfloat16, 1.0, 310, "cuda", t) for t in range(3))
    pats = [(N, r)] * (1 if H == 17 else 4)
    compare_full(q, k, v, pats, True, "bf16", tag=f"wide H{H}", heads=[0, H - 1])


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("causal,lost", [(True, (32, 64)), (True, (1, 64)), (True, (64, 128)), (False, (0, 32)),
                                         (False, (32, 64)), (False, (0, 64)), (False, (0, 199))], ids=str)
@pytest.mark.parametrize("H,offset", [(2, 0.0), (2, 32.0), (260, 0.0)])
def test_scores_overflowing_to_minus_infinity(H, offset, causal, lost, D):
    """q.k of the keys `lost` is -2^140, minus infinity in float32 and without
    weight in the oracle: a wave that sees only such keys in its first block (or
    the row's first tile) leaves the row to the others, with 2 heads (split
    keys) and with 260 (two items of 128 rows each: 520 of them).  `offset`
    raises the finite scores (about 370 in log2 units at D = 64): the reference
    max is found again once a finite score is seen."""
    N = 200
    note(f"[split] -inf keys {lost} H={H} D={D} causal={causal} offset={offset}")
    q, k, v = (workloads.make_random((1, N, H, D), torch.bfloat16, 1.0, 320 + D, "cuda", t) for t in range(3))
    q[..., 0], k[..., 0] = 2.0 ** 70, 0.0
    k[:, lost[0]:lost[1], :, 0] = -(2.0 ** 70)
    if offset:
        q[..., 1], k[..., 1] = 64.0, offset
    compare_full(q, k, v, [(N, 1)], causal, "bf16", tag=f"-inf {lost} H{H} D{D}", heads=[0, H - 1])


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("H", [2, 260])
def test_scores_far_below_zero(H, causal, D):
    """Every score about -2048 / sqrt(D): the first tile's reference max lies
    below -128 in log2 units, whose negative has no float32 power of two."""
    note(f"[split] low scores H={H} D={D} causal={causal}")
    q, k, v = (workloads.make_random((1, 200, H, D), torch.bfloat16, 1.0, 330 + D, "cuda", t) for t in range(3))
    q[..., 1], k[..., 1] = 64.0, -32.0
    compare_full(q, k, v, [(200, 1), (100, 2)], causal, "bf16", tag=f"low H{H} D{D}", heads=[0, H - 1])


@pytest.mark.parametrize("D", [32, 64, 128])
def test_a_sequence_alone_and_in_a_batch(D):
    """Float32 gives the same bits; bf16 may take the other form in the batch,
    whose results differ within the bars both keep to the oracle (2e-2 on out
    and 1e-2 on lse, twice).  The backward, given the same out and lse, gives
    the same bits."""
    from paper_2307_02486_amd import dilated_attn, dilated_attn_bwd
    note(f"[split] batch D={D}")
    pats = [(300, 1), (700, 2)]
    for dtype in (torch.float32, torch.bfloat16):
        q, k, v, dout = (workloads.make_random((16, 700, 8, D), dtype, 1.0, 340, "cuda", t) for t in range(4))
        out, lse = dilated_attn(q, k, v, pats)
        one, l1 = dilated_attn(q[:1], k[:1], v[:1], pats)
        if dtype == torch.float32:
            assert torch.equal(one, out[:1]) and torch.equal(l1, lse[:1])
            continue
        assert float((one.float() - out[:1].float()).abs().max()) <= 4e-2
        assert float((l1 - lse[:1]).abs().max()) <= 2e-2
        grads = dilated_attn_bwd(q, k, v, out, lse, dout, pats)
        alone = dilated_attn_bwd(q[:1], k[:1], v[:1], out[:1], lse[:1], dout[:1], pats)
        assert all(torch.equal(a, g[:1]) for a, g in zip(alone, grads))
