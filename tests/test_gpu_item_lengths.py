"""Items of every length at which the step sequence takes another way: one block to one round of a ring and
over, and both sides of the groups of 64 block ids, against the oracle; rows whole, so that a row is an item."""

import numpy as np
import pytest
import torch

import paper_2511_23113_amd as dbsp
from oracle import attention as oa
from paper_2511_23113_amd.binding import ITEMS

O_TOL, LSE_TOL = 1e-2, 1e-3          # bf16 inputs and probabilities, f32 sums, |O| <= 1
# O of a long row is the mean of many values and small, so that a wrong slice of V hides in an absolute tolerance: each
# query block's O is held against its own size too (2-norms).  Probabilities and O are each rounded to bf16, by 2^-9
# at most of their value; the probabilities' roundings are independent from key to key, as V's values are, so they add up
# as the products themselves do: at most sqrt(2) 2^-9 = 2.8e-3 together.  32 wrong keys of 16,768 are 4e-2.
O_REL_TOL = 5e-3
LENGTHS = [1, 2, 3, 4, 5, 6, 7, 8, 9, 63, 64, 65, 66, 67, 127, 128, 129, 131]
KERNELS = [(64, 64, False), (128, 64, False), (64, 128, False), (128, 128, False), (64, 128, True)]


def masks_by_length(block, d, pair, P):
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
    return rows, mask


def rel_errors(got, ref, block):
    """2-norm of the difference over the 2-norm of the result, query block by query block."""
    got, ref = (np.asarray(x, np.float64).reshape(-1, block * x.shape[-1]) for x in (got, ref))
    return np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)


@pytest.mark.gpu
@pytest.mark.parametrize("block,d,pair", KERNELS)
@pytest.mark.parametrize("P", [1, 7])                # one workgroup walks all items one behind the other, or seven share them
@pytest.mark.parametrize("mode", [dbsp.MODE_BALANCED, dbsp.MODE_ROUNDS])       # kernels differ in how long a barrier waits
def test_item_lengths(block, d, pair, P, mode):
    _, mask = masks_by_length(block, d, pair, P)
    _, nQ, nK = mask.shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(P)
    q, k = (torch.randn((1, 1, n * block, d), generator=gen, device="cuda").to(torch.bfloat16) for n in (nQ, nK))
    v = (2 * torch.rand((1, 1, nK * block, d), generator=gen, device="cuda") - 1).to(torch.bfloat16)
    plan = dbsp.plan_sparse_attn(mask, block, num_partitions=P, max_item_len=nK, pair_rows=pair, mode=mode)
    assert sorted(np.asarray(plan.array(ITEMS)).reshape(-1, 4)[:, 3].tolist()) == sorted(LENGTHS)
    ref_o, ref_l = oa.masked_attention(*(x.float().cpu().numpy() for x in (q, k, v)), mask, block, dtype=np.float32)
    for _ in range(2):
        o, lse = torch.full_like(q, float("nan")), torch.full((1, 1, nQ * block), float("nan"), device="cuda")
        dbsp.sparse_attn_fwd(plan, q, k, v, o=o, lse=lse)
        torch.cuda.synchronize()
        got_o = o.float().cpu().numpy()
        assert np.abs(got_o - ref_o).max() <= O_TOL
        assert rel_errors(got_o, ref_o, block).max() <= O_REL_TOL
        assert np.abs(lse.cpu().numpy() - ref_l).max() <= LSE_TOL
    plan.close()


@pytest.mark.parametrize("block,d,pair", KERNELS)
def test_one_wrong_slice_of_v_is_seen_at_every_length(block, d, pair):
    # (in the oracle: the item's last block, or 32 keys of it, hold another block's values)
    rows, mask = masks_by_length(block, d, pair, 1)
    nK = mask.shape[2]
    rng = np.random.default_rng(1)
    gen = torch.Generator().manual_seed(1)
    q, k = (torch.randn((1, 1, n * block, d), generator=gen).to(torch.bfloat16).float().numpy() for n in (mask.shape[1], nK))
    v = (2 * torch.rand((1, 1, nK * block, d), generator=gen) - 1).to(torch.bfloat16).float().numpy()
    per_item = 2 if pair else 1
    ref, _ = oa.masked_attention(q, k, v, mask, block, dtype=np.float32)
    ref = ref.reshape(len(rows), per_item, -1, d)
    for i, n in enumerate(rows):
        own = mask[0, per_item * i:per_item * (i + 1)].any(axis=0).nonzero()[0]
        last, other = own[-1], rng.choice(np.setdiff1d(np.arange(nK), own[-1:]))
        for lo, hi in ((0, block), (block - 32, block)):
            wrong = v.copy()
            wrong[0, 0, last * block + lo:last * block + hi] = v[0, 0, other * block + lo:other * block + hi]
            got, _ = oa.masked_attention_rows(q, k, wrong, mask, block, [(0, 0, per_item * i + y) for y in range(per_item)], dtype=np.float32)
            assert rel_errors(got, ref[i], block).max() > 2 * O_REL_TOL, (n, lo)


@pytest.mark.gpu
@pytest.mark.parametrize("block,d,pair", [(128, 128, False), (64, 128, True)])
@pytest.mark.parametrize("P", [1, 7])
def test_item_lengths_under_a_placement_without_locality(block, d, pair, P):         # the kernels of the shorter wait
    test_item_lengths(block, d, pair, P, dbsp.MODE_NAIVE)


@pytest.mark.gpu
@pytest.mark.parametrize("block, d, pair", [(128, 128, False), (128, 64, False), (64, 128, True), (64, 64, False)])
@pytest.mark.parametrize("offset", [1, 2, 4, 8])
def test_queries_at_any_address(block, d, pair, offset):
    # Q goes through the LDS where its address is a multiple of 16 bytes, else straight to registers: the same bits
    H, nQ, nK = 2, 5, 7
    rng = np.random.default_rng(offset)
    mask = (rng.random((H, nQ, nK)) < 0.6).astype(np.uint8)
    q = torch.randn((1, H, nQ * block, d), device="cuda").to(torch.bfloat16)
    k, v = (torch.randn((1, H, nK * block, d), device="cuda").to(torch.bfloat16) for _ in range(2))
    moved = torch.empty(q.numel() + offset, device="cuda", dtype=torch.bfloat16)[offset:].view(q.shape)
    moved.copy_(q)
    for kw in (dict(num_partitions=2), dict(num_partitions=3, mode=dbsp.MODE_ROUNDS, dynamic_tail=400), dict(num_partitions=64, max_item_len=2)):
        plan = dbsp.plan_sparse_attn(mask, block, pair_rows=pair, **kw)
        o, lse = dbsp.sparse_attn_fwd(plan, q, k, v)
        om, lsem = dbsp.sparse_attn_fwd(plan, moved, k, v, o=torch.empty_like(q), lse=torch.empty_like(lse))
        assert torch.equal(o, om) and torch.equal(lse, lsem)
