"""Greedy placements run their partitions' items longest first and give every compute die partitions in a row: which
workgroup runs what, at partition counts with and without whole runs for every die, against the same items placed naively
(an item's result does not depend on who computes it, and a split row's chunks are merged in their own order: the outputs
are the same bits) and against the oracle."""

import numpy as np
import pytest

import synth
from oracle import attention as oa

pytestmark = pytest.mark.gpu

O_TOL, LSE_TOL = 1e-2, 1e-3


def _run(plan, q, k, v):
    import torch
    import paper_2511_23113_amd as dbsp
    o, lse = dbsp.sparse_attn_fwd(plan, q, k, v)
    torch.cuda.synchronize()
    return o.float().cpu().numpy(), lse.cpu().numpy()


# 60 rows of up to 13 blocks, too few for runs on the dies: equal rows, rows of all lengths, empty rows (workgroups behind the
# last partition that has items); with 64-token blocks the items are too short for an order of their own
@pytest.mark.parametrize("block, d", [(128, 128), (64, 64)])
@pytest.mark.parametrize("kind", ["equal", "ragged", "empty_rows"])
@pytest.mark.parametrize("P", [7, 8, 15, 16, 33, 60, 64, 130, 256])
def test_every_partition_runs_once(block, d, kind, P):
    import paper_2511_23113_amd as dbsp
    from paper_2511_23113_amd import binding as B
    from test_gpu_attention import _dev
    H, nQ, nK = 3, 20, 13
    rng = np.random.default_rng(P)
    keep = {"equal": np.full((H, nQ), 9), "ragged": rng.integers(1, nK + 1, (H, nQ)), "empty_rows": rng.integers(0, 2, (H, nQ)) * 9}[kind]
    mask = np.zeros((H, nQ, nK), np.uint8)
    for h in range(H):
        for i in range(nQ):
            mask[h, i, rng.permutation(nK)[:keep[h, i]]] = 1
    qb, kb, vb = (synth.normal_bf16((1, H, n * block, d), s) for n, s in ((nQ, 1), (nK, 2), (nK, 3)))
    q, k, v = _dev(qb), _dev(kb), _dev(vb)
    greedy = dbsp.plan_sparse_attn(mask, block, num_partitions=P, max_item_len=9)
    o, lse = _run(greedy, q, k, v)
    ticks, _ = greedy.busy()
    assert np.array_equal(ticks > 0, greedy.array(B.PART_LOAD) > 0)          # a partition's time is its own
    o0, lse0 = _run(dbsp.plan_sparse_attn(mask, block, num_partitions=P, max_item_len=9, mode=dbsp.MODE_NAIVE), q, k, v)
    assert np.array_equal(o, o0) and np.array_equal(lse, lse0)
    kept, _, _ = dbsp.plan_sparse_attn_reuse(greedy, mask, 8.0, max_item_len=9)
    o1, lse1 = _run(kept, q, k, v)
    assert np.array_equal(o, o1) and np.array_equal(lse, lse1)
    if P in (8, 60):
        Or, Lr = oa.masked_attention(*(synth.bf16_bits_to_f32(x) for x in (qb, kb, vb)), mask, block)
        some = ~np.isneginf(Lr)
        assert np.array_equal(~np.isneginf(lse), some)
        assert np.abs(o - Or).max() <= O_TOL * max(1.0, np.abs(Or).max()) and np.abs(lse[some] - Lr[some]).max() <= LSE_TOL


# Partitions in runs on the dies, with and without some behind the last whole runs, lists sorted one by one (equal rows: two items
# for the first partitions, one for the others) and by counting (rows of all lengths, ten a partition)
@pytest.mark.parametrize("block, d, pair", [(128, 128, False), (128, 64, False), (64, 64, False), (64, 128, False), (64, 128, True)])
@pytest.mark.parametrize("kind", ["equal", "ragged"])
@pytest.mark.parametrize("P, twos", [(64, 32), (127, 64), (200, 96), (256, 128)])
def test_partitions_in_runs(block, d, pair, kind, P, twos):
    import torch
    import paper_2511_23113_amd as dbsp
    from paper_2511_23113_amd import binding as B
    rows = P + twos if kind == "equal" else 10 * P
    per, nK = (2, 80) if pair else (1, 40)
    rng = np.random.default_rng(P)
    keep = np.full(rows, 17) if kind == "equal" else rng.integers(17, 41, rows)
    mask = np.zeros((1, rows * per, nK), np.uint8)
    for i in range(rows):
        mask[0, per * i:per * i + per, rng.permutation(nK)[:keep[i] * per]] = 1
    q, k, v = (torch.randn((1, 1, n * block, d), device="cuda").to(torch.bfloat16) for n in (rows * per, nK, nK))

    def launched(plan):
        o = torch.full_like(q, float("nan"))
        lse = torch.full(q.shape[:3], float("nan"), device="cuda")
        for _ in range(2):
            dbsp.sparse_attn_fwd(plan, q, k, v, o=o, lse=lse)
        torch.cuda.synchronize()
        return o, lse

    kw = dict(num_partitions=P, max_item_len=-1, pair_rows=pair)
    greedy = dbsp.plan_sparse_attn(mask, block, **kw)
    of = greedy.run_order()["partition_of"]
    assert not np.array_equal(of, np.arange(P)) and sorted(of) == list(range(P))
    want = launched(dbsp.plan_sparse_attn(mask, block, mode=dbsp.MODE_NAIVE, **kw))
    assert bool(torch.isfinite(want[0]).all()) and bool(torch.isfinite(want[1]).all())
    kept, reused, _ = dbsp.plan_sparse_attn_reuse(greedy, mask, 8.0, max_item_len=-1)
    assert reused
    for plan in (greedy, kept):
        got = launched(plan)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        ticks, hw = plan.busy()
        for die in range(8):                                  # times and places are their partitions' own
            assert len(set(hw[of[die::8]] >> 16)) == 1
        if kind == "equal":
            two = np.diff(plan.array(B.PART_PTR)) == 2
            assert two.sum() == twos and ticks[two].min() > 1.2 * np.median(ticks[~two])


# 60 rows and a mask that leaves their partitions dealt one by one; 600 equal rows, dealt in runs as with costs; 600 of all lengths
@pytest.mark.parametrize("block, d", [(128, 128), (64, 64)])
@pytest.mark.parametrize("rows", [60, 600])
@pytest.mark.parametrize("P", [64, 130, 256])
@pytest.mark.parametrize("kind", ["equal", "ragged"])
def test_costs_stay_with_the_compute_unit(block, d, rows, P, kind):
    import paper_2511_23113_amd as dbsp
    import torch
    from oracle import planner as op
    from paper_2511_23113_amd import binding as B
    H, nQ, nK = 3, rows // 3, 40
    rng = np.random.default_rng(P)
    keep = np.full((H, nQ), 21) if kind == "equal" else rng.integers(17, nK + 1, (H, nQ))
    mask = np.zeros((H, nQ, nK), np.uint8)
    for h in range(H):
        for i in range(nQ):
            mask[h, i, rng.permutation(nK)[:keep[h, i]]] = 1
    q, k, v = (torch.randn((1, H, n * block, d), device="cuda").to(torch.bfloat16) for n in (nQ, nK, nK))

    def launched(**kw):
        plan = dbsp.plan_sparse_attn(mask, block, num_partitions=P, max_item_len=-1, **kw)
        dbsp.sparse_attn_fwd(plan, q, k, v)
        return (plan, *plan.busy())

    plain, ticks, hw = launched()
    cost = plain.calibrate()
    by_partition = np.asarray(op.calibrate_cost(ticks.tolist(), plain.array(B.PART_LOAD).tolist()))
    tuned, ticks, hw_tuned = launched(partition_cost=cost)
    # where a plan of more items than partitions runs them
    there = dbsp.plan_sparse_attn(np.ones((1, 2 * P, 1), np.uint8), block, partition_cost=cost, host_only=True).run_order()["partition_of"]
    here, now = (plan.run_order()["partition_of"] for plan in (plain, tuned))
    assert np.array_equal(cost[there], by_partition[here])
    # workgroup b is on one die in every launch
    both = (plain.array(B.PART_LOAD)[here] > 0) & (tuned.array(B.PART_LOAD)[now] > 0)
    assert both.any() and np.array_equal(hw[here][both] >> 16, hw_tuned[now][both] >> 16)
    if rows > P:
        assert np.array_equal(now, there)
    assert tuned.calibrate()[there].tolist() == np.asarray(op.calibrate_cost(ticks.tolist(), tuned.array(B.PART_LOAD).tolist()))[now].tolist()
