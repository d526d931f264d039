"""What the workgroups of a launch run, and in what order, on the host: the greedy placement's lists longest first and its
partitions in runs on a die, against the rule worked out from the plan's own arrays; with costs, one and the same
workgroup for a partition whatever the mask."""

import numpy as np
import pytest

import paper_2511_23113_amd as dbsp
from paper_2511_23113_amd import binding as B

DIES = 8


def dealt(n, lg, P):
    """Partitions by workgroup: runs of 2^lg partitions dealt to the dies in turn, die x's workgroups being x, x + 8, ..."""
    size = 1 << lg
    whole = n // (DIES * size) * (DIES * size)
    of = np.arange(P)
    for die in range(DIES):
        runs = [g for k in range(die, whole // size, DIES) for g in range(k * size, (k + 1) * size)]
        of[die:whole:DIES] = runs
    return of


def longest_runs(n):
    return max(lg for lg in range(1, 32) if DIES << lg <= n) if n >= 64 else 0


def runs_of(load):
    """log2 of the longest runs by which no die has over 3 % more blocks than the mean: load of the partitions in use."""
    for lg in range(longest_runs(len(load)), 0, -1):
        of = dealt(len(load), lg, len(load))
        if max(100 * DIES * int(load[of[die::DIES]].sum()) for die in range(DIES)) <= 103 * int(load.sum()):
            return lg
    return 0


def mask_of(rows, nK, seed):
    """One head, row i with rows[i] active blocks."""
    rng = np.random.default_rng(seed)
    mask = np.zeros((1, len(rows), nK), np.uint8)
    for i, n in enumerate(rows):
        mask[0, i, rng.permutation(nK)[:n]] = 1
    return mask


def lists(plan, items):
    """Items of every workgroup, in the order they run."""
    order = plan.run_order()
    of, run = order["partition_of"], order["items"]
    ptr, n = plan.array(B.PART_PTR), np.diff(plan.array(B.PART_PTR))
    ends = np.cumsum(n[of])
    own = [run[e - c:e] for e, c in zip(ends, n[of])]
    placed = plan.array(B.PART_ITEMS)
    for b, mine in enumerate(own):
        assert sorted(mine) == sorted(placed[ptr[of[b]]:ptr[of[b] + 1]])
    assert sorted(run) == list(range(len(items)))
    return of, own


ROWS = {                               # of up to 40 blocks
    "equal": lambda rng, n: np.full(n, 9),
    "ragged": lambda rng, n: rng.integers(1, 41, n),
    "empty": lambda rng, n: rng.integers(0, 2, n) * 17,
    "short": lambda rng, n: rng.integers(1, 4, n),
}


@pytest.mark.parametrize("P", [1, 7, 8, 63, 64, 65, 127, 128, 130, 200, 223, 224, 256, 512, 1024])
@pytest.mark.parametrize("kind", list(ROWS))
@pytest.mark.parametrize("block, pair", [(128, False), (64, False), (64, True)])
def test_every_partition_runs_once_longest_first(P, kind, block, pair):
    rng = np.random.default_rng(P)
    for n in (5, 90, 223, 224, 700, 3000):
        mask = mask_of(ROWS[kind](rng, n) * (1 if block == 128 or pair else 3), 128, n)
        plan = dbsp.plan_sparse_attn(mask, block, num_partitions=P, max_item_len=60, pair_rows=pair, host_only=True)
        items, load = plan.array(B.ITEMS).reshape(-1, 4), plan.array(B.PART_LOAD)
        of, own = lists(plan, items)
        used = max([g + 1 for g in range(P) if plan.array(B.PART_PTR)[g + 1] > plan.array(B.PART_PTR)[g]], default=0)
        length = items[:, 3] - items[:, 2]
        rows = 128 if pair else block
        worth = length.sum() * rows * rows >= 4 * 128 * 128 * len(length)
        assert np.array_equal(of, dealt(used, runs_of(load[:used]) if worth else 0, P))
        # an item each: nothing to put in an order, which shows where they fill the chip
        assert plan.run_order()["local"] == (max(map(len, own)) > 1 or used < 224)
        for mine in own:
            assert list(mine) == (sorted(mine, key=lambda i: (-length[i], i)) if worth else sorted(mine))


def test_other_placements_run_as_they_stand():
    mask = mask_of(ROWS["ragged"](np.random.default_rng(0), 700), 64, 0)
    for kw in (dict(mode=B.MODE_NAIVE), dict(mode=B.MODE_ROUNDS, locality_groups=8), dict(mode=B.MODE_ROUNDS, dynamic_tail=40),
               dict(mode=B.MODE_REWARD, locality_groups=8, reward=1.0), dict(mode=B.MODE_ROUNDS, partition_cost=np.arange(1, 257))):
        plan = dbsp.plan_sparse_attn(mask, 128, num_partitions=256, host_only=True, **kw)
        order = plan.run_order()
        assert np.array_equal(order["partition_of"], np.arange(256)) and np.array_equal(order["items"], plan.array(B.PART_ITEMS))
        assert order["local"] == (kw["mode"] == B.MODE_ROUNDS)


@pytest.mark.parametrize("P", [7, 64, 130, 256, 1024])
def test_with_costs_a_partitions_workgroup_is_settled_by_their_number(P):
    rng = np.random.default_rng(P)
    cost = rng.integers(950, 1100, P).astype(np.int32)
    for kind in ROWS:
        for n in (5, 90, 700, 3000):
            mask = mask_of(ROWS[kind](rng, n), 64, n)
            plan = dbsp.plan_sparse_attn(mask, 128, partition_cost=cost, max_item_len=30, host_only=True)
            of, own = lists(plan, plan.array(B.ITEMS).reshape(-1, 4))
            if max(map(len, own)) > 1:
                assert np.array_equal(of, dealt(P, longest_runs(P), P))
            else:                       # an item each, whatever the costs: as without
                plain = dbsp.plan_sparse_attn(mask, 128, num_partitions=P, max_item_len=30, host_only=True)
                assert np.array_equal(of, plain.run_order()["partition_of"])
            # a placement carried over stays where it is
            kept, reused, _ = dbsp.plan_sparse_attn_reuse(plan, mask, 1e9, max_item_len=30, host_only=True)
            assert reused and np.array_equal(kept.run_order()["partition_of"], of)
