"""Scores that are not finite, on the GPU.  Keys masked by scores of -inf have probability 0, wherever they lie in a
block (against the oracle); a query with an undefined score has NaN as its O and LSE, and no other query has."""

import numpy as np
import pytest
import torch

import paper_2511_23113_amd as dbsp
from oracle import attention as oa

pytestmark = pytest.mark.gpu

O_TOL, LSE_TOL = 1e-2, 1e-3          # bf16 inputs and probabilities, f32 sums, |O| <= 1


@pytest.mark.parametrize("block,d", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("which", ["first 32 keys", "last 32 keys", "a block", "all"])
@pytest.mark.parametrize("scale,length", [(0.0, -1), (0.0, 2), (3.0, -1)])      # plan rows whole, cut; a scale at which the lowest float overflows
def test_masked_keys(block, d, which, scale, length):
    H, n = 2, 5
    rng = np.random.default_rng(block + d)
    mask = (rng.random((H, n, n)) < 0.6).astype(np.uint8)
    mask[:, range(n), range(n)] = 1
    mask[:, :, 4] = 1                    # every row has a block beside block 0
    gen = torch.Generator(device="cuda")
    gen.manual_seed(block)
    q, k = (torch.randn((1, H, n * block, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    v = (2 * torch.rand((1, H, n * block, d), generator=gen, device="cuda") - 1).to(torch.bfloat16)
    pos = torch.arange(n * block, device="cuda")
    masked = {"first 32 keys": pos % block < 32, "last 32 keys": pos % block >= block - 32, "a block": pos < block, "all": pos >= 0}[which]
    q[..., 0] = 1
    k[:, :, masked, 0] = float("-inf")
    with np.errstate(invalid="ignore"):
        ref_o, ref_l = oa.masked_attention(*(x.float().cpu().numpy() for x in (q, k, v)), mask, block, scale=scale or None)
    plan = dbsp.plan_sparse_attn(mask, block, max_item_len=length, num_partitions=16)
    o, lse = dbsp.sparse_attn_fwd(plan, q, k, v, softmax_scale=scale)
    torch.cuda.synchronize()
    got_o, got_l = o.float().cpu().numpy(), lse.cpu().numpy()
    if which == "all":                   # nothing left to weigh: 0 / 0
        assert np.isnan(got_o).all() and np.isneginf(got_l).all()
        return
    assert np.abs(got_o - ref_o).max() <= O_TOL
    assert np.abs(got_l - ref_l).max() <= LSE_TOL


@pytest.mark.parametrize("block,d,pair", [(64, 64, False), (64, 128, False), (128, 64, False), (128, 128, False), (64, 128, True)])
@pytest.mark.parametrize("length", [-1, 2, 1])          # rows whole, cut, cut into single blocks
@pytest.mark.parametrize("which", ["a key", "a query", "an infinite score"])
def test_undefined_scores_show(block, d, pair, length, which):
    H, n, key, query = 2, 6, 37, 5
    rng = np.random.default_rng(block + d)
    mask = (rng.random((H, n, n)) < 0.6).astype(np.uint8)
    mask[:, range(n), range(n)] = 1
    mask[1, 4:] = 0                      # rows that are empty
    gen = torch.Generator(device="cuda")
    gen.manual_seed(block)
    q, k, v = (torch.randn((1, H, n * block, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    nan = torch.zeros((H, n * block), dtype=torch.bool)
    rows = torch.from_numpy(mask).bool().repeat_interleave(block, 1)          # [H, queries, KV blocks]
    if which == "a query":
        q[0, :, query] = float("nan")
        nan[:, query] = True
    else:                                # in KV block 2
        if which == "a key":
            k[0, :, 2 * block + key] = float("nan")
        else:                            # inf - inf where the running max reaches it
            q[..., 0] = 1
            k[0, :, 2 * block + key, 0] = float("inf")
        nan |= rows[:, :, 2]
        if pair:                         # computed for both query blocks of a pair, and documented as undefined there
            nan |= rows[:, :, 2].reshape(H, n // 2, 2, block).any(2, keepdim=True).expand(-1, -1, 2, -1).reshape(H, -1)
    plan = dbsp.plan_sparse_attn(mask, block, max_item_len=length, num_partitions=16, pair_rows=pair)
    o, lse = dbsp.sparse_attn_fwd(plan, q, k, v)
    torch.cuda.synchronize()
    o, lse = o[0].float().cpu(), lse[0].cpu()
    if pair and which != "a query":      # (undefined where only the neighbour needs the block)
        sure = rows[:, :, 2]
        assert lse[sure].isnan().all() and o[sure].isnan().all()
        assert not lse[~nan].isnan().any() and not o[~nan].isnan().any()
        return
    assert torch.equal(lse.isnan(), nan)
    assert torch.equal(o.isnan(), nan[..., None].expand_as(o))
