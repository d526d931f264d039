"""Split rows on the GPU: merged in place by the kernel's waves or by a launch behind it, on both sides of the
rule that picks, against the oracle.  P partitions and max_item_len choose the side: in place while there are no
more items than partitions and a wave's share of a row is at most 14 tiles (4 tiles a chunk at d = 128; at d = 64
2 with 64-token and 1 with 128-token blocks)."""

import numpy as np
import pytest
import torch

import paper_2511_23113_amd as dbsp
from oracle import attention as oa

pytestmark = pytest.mark.gpu

O_TOL, LSE_TOL = 1e-2, 1e-3          # bf16 inputs and probabilities, f32 sums, |O| <= 1


@pytest.mark.parametrize("block,d,pair,length", [
    (64, 64, False, 2), (64, 64, False, 3), (64, 64, False, 5),          # 7 to 20 chunks of rows of 20 blocks
    (128, 64, False, 1), (128, 64, False, 2), (128, 64, False, 9),
    (64, 128, False, 5), (64, 128, False, 7), (64, 128, False, 10),
    (128, 128, False, 1), (128, 128, False, 5), (128, 128, False, 7),
    (64, 128, True, 2), (64, 128, True, 3), (64, 128, True, 4),
])
@pytest.mark.parametrize("P", [8, 1024])
def test_both_ways_to_merge(block, d, pair, length, P):
    rng = np.random.default_rng(block + d + length)
    B, H, nQ, nK = 2, 2, 5, 20
    mask = (rng.random((H, nQ, nK)) < 0.6).astype(np.uint8)
    mask[0, 0] = 1                       # a full row, one of a single block, an empty one
    mask[0, 1] = 0
    mask[0, 1, 7] = 1
    mask[1, 2] = 0
    gen = torch.Generator(device="cuda")
    gen.manual_seed(length)
    q, k = (torch.randn((B, H, n * block, d), generator=gen, device="cuda").to(torch.bfloat16) for n in (nQ, nK))
    v = (2 * torch.rand((B, H, nK * block, d), generator=gen, device="cuda") - 1).to(torch.bfloat16)
    plan = dbsp.plan_sparse_attn(mask, block, num_partitions=P, max_item_len=length, max_batch=B, pair_rows=pair)
    ref_o, ref_l = oa.masked_attention(*(x.float().cpu().numpy() for x in (q, k, v)), mask, block)
    empty = np.isneginf(ref_l)
    for _ in range(3):                   # counters and scratch are left ready for the next launch
        o, lse = torch.full_like(q, float("nan")), torch.full((B, H, nQ * block), float("nan"), device="cuda")
        dbsp.sparse_attn_fwd(plan, q, k, v, o=o, lse=lse)
        torch.cuda.synchronize()
        got_o, got_l = o.float().cpu().numpy(), lse.cpu().numpy()
        assert np.abs(got_o - ref_o).max() <= O_TOL
        assert np.array_equal(np.isneginf(got_l), empty)
        assert np.abs(got_l[~empty] - ref_l[~empty]).max() <= LSE_TOL
    plan.close()
