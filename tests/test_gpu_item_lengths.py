"""Items of every length at which the step sequence takes another way: one block to one round of a ring and
over, and both sides of the groups of 64 block ids, against the oracle; rows whole, so that a row is an item."""

import numpy as np
import pytest
import torch

import paper_2511_23113_amd as dbsp
from oracle import attention as oa
from paper_2511_23113_amd.binding import ITEMS

pytestmark = pytest.mark.gpu

O_TOL, LSE_TOL = 1e-2, 1e-3          # bf16 inputs and probabilities, f32 sums, |O| <= 1
LENGTHS = [1, 2, 3, 4, 5, 6, 7, 8, 9, 63, 64, 65, 66, 67, 127, 128, 129, 131]


@pytest.mark.parametrize("block,d,pair", [(64, 64, False), (128, 64, False), (64, 128, False), (128, 128, False), (64, 128, True)])
@pytest.mark.parametrize("P", [1, 7])                # one workgroup walks all items one behind the other, or seven share them
def test_item_lengths(block, d, pair, P):
    rng = np.random.default_rng(block + d + P)
    nK = 131 * (2 if pair else 1)                    # pair rows: an item's length is in pairs of KV blocks
    rows = rng.permutation(LENGTHS)
    mask = np.zeros((1, len(rows) * (2 if pair else 1), nK), np.uint8)
    for i, n in enumerate(rows):
        if pair:                                     # both query blocks together have 2 n blocks, unlike ones
            own = rng.permutation(nK)[:2 * n]
            mask[0, 2 * i, own[: n + n // 2]] = 1
            mask[0, 2 * i + 1, own[n // 2:]] = 1
        else:
            mask[0, i, rng.permutation(nK)[:n]] = 1
    nQ = mask.shape[1]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(P)
    q, k = (torch.randn((1, 1, n * block, d), generator=gen, device="cuda").to(torch.bfloat16) for n in (nQ, nK))
    v = (2 * torch.rand((1, 1, nK * block, d), generator=gen, device="cuda") - 1).to(torch.bfloat16)
    plan = dbsp.plan_sparse_attn(mask, block, num_partitions=P, max_item_len=nK, pair_rows=pair)
    assert sorted(np.asarray(plan.array(ITEMS)).reshape(-1, 4)[:, 3].tolist()) == sorted(LENGTHS)
    ref_o, ref_l = oa.masked_attention(*(x.float().cpu().numpy() for x in (q, k, v)), mask, block, dtype=np.float32)
    for _ in range(2):
        o, lse = torch.full_like(q, float("nan")), torch.full((1, 1, nQ * block), float("nan"), device="cuda")
        dbsp.sparse_attn_fwd(plan, q, k, v, o=o, lse=lse)
        torch.cuda.synchronize()
        assert np.abs(o.float().cpu().numpy() - ref_o).max() <= O_TOL
        assert np.abs(lse.cpu().numpy() - ref_l).max() <= LSE_TOL
    plan.close()
