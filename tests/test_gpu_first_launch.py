"""Small plans' first launches read the plan where it is staged once their device buffer has been a plan's before: new
masks call after call, each plan launched once or several times, on one stream or another, against the same items' results
from a plan that another buffer's first launch has fetched."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# split rows (counters), rows that are not split, empty rows, an item for every workgroup and for few of them
@pytest.mark.parametrize("block, d", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("length", [2, 4, -1])
@pytest.mark.parametrize("mode", [0, 2])
def test_first_launches_of_small_plans(block, d, length, mode):
    import torch
    import paper_2511_23113_amd as dbsp
    H, nQ, nK = 2, 6, 7
    rng = np.random.default_rng(block + d + length)
    gen = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn((1, H, n * block, d), generator=gen, device="cuda").to(torch.bfloat16) for n in (nQ, nK, nK))
    streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    staged = 0
    for step in range(24):
        mask = (rng.random((H, nQ, nK)) < rng.choice([0.1, 0.4, 0.8])).astype(np.uint8)
        mask[0, 0, 0] = 1
        kw = dict(max_item_len=length, mode=mode, num_partitions=int(rng.choice([64, 256])))
        # one partition: more than an item a workgroup, which is fetched
        want_o, want_lse = dbsp.sparse_attn_fwd(dbsp.plan_sparse_attn(mask, block, max_item_len=length, num_partitions=1), q, k, v)
        torch.cuda.synchronize()
        plan = dbsp.plan_sparse_attn(mask, block, **kw)
        for launch in range(1 + step % 3):
            with torch.cuda.stream(streams[(step + launch) % 2]):
                o, lse = dbsp.sparse_attn_fwd(plan, q, k, v)
            if launch % 2 == 0:
                torch.cuda.synchronize()      # (a plan's calls do not overlap)
            else:
                streams[(step + launch) % 2].synchronize()
            # merged two chunks at a time here, four there: a rounding of O apart, a few of LSE (at most 8)
            torch.testing.assert_close(o, want_o, rtol=2.0 ** -7, atol=1e-4)
            torch.testing.assert_close(lse, want_lse, rtol=0, atol=8 * 2.0 ** -21)
            # and the same bits from launch to launch, whichever way the plan was read
            if launch == 0:
                first_o, first_lse = o, lse
            assert torch.equal(o, first_o) and torch.equal(lse, first_lse)
        ticks, _ = plan.busy()
        assert mode == 2 or np.array_equal(ticks > 0, plan.array(7) > 0)          # 7: blocks per partition
        staged += plan.run_order()["staged"]
        del plan
    assert staged > 0


def test_a_batch_or_the_static_scratch_fetches():
    import torch
    import paper_2511_23113_amd as dbsp
    rng = np.random.default_rng(5)
    q, k, v = (torch.randn((2, 2, 6 * 64, 64), device="cuda").to(torch.bfloat16) for _ in range(3))
    for step in range(12):
        mask = (rng.random((2, 6, 6)) < 0.6).astype(np.uint8)
        plan = dbsp.plan_sparse_attn(mask, 64, max_item_len=2, max_batch=2)
        outs = []
        for call in ((0, 1), (1, 0), (0, 0))[step % 3]:
            if call:
                outs.append(dbsp.sparse_attn_fwd(plan, q, k, v)[0][:1])
            else:
                outs.append(dbsp.sparse_attn_fwd(plan, q[:1], k[:1], v[:1], static_scratch=step % 2 == 0)[0])
        torch.cuda.synchronize()
        torch.testing.assert_close(outs[0], outs[1], rtol=2.0 ** -7, atol=1e-4)        # (merged in place or behind the launch)


def test_a_capture_right_behind_a_first_launch():
    """The captured call sends the plan on the library's own stream while the first launch is yet to run (behind a long
    kernel), runs or has just ended: its results and busy times, every replay and the buffer's next plans stay right."""
    import torch
    import paper_2511_23113_amd as dbsp
    H, n, block, d = 2, 8, 64, 64
    rng = np.random.default_rng(7)
    gen = torch.Generator(device="cuda").manual_seed(7)
    q, k, v = (torch.randn((1, H, n * block, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    masks = [(rng.random((H, n, n)) < 0.7).astype(np.uint8) for _ in range(3)]
    wants = []
    for mask in masks:
        plan = dbsp.plan_sparse_attn(mask, block)
        assert len(plan.array(4)) > 0                              # 4: split rows
        for _ in range(2):                                         # the second launch is of the fetched plan
            wants.append(dbsp.sparse_attn_fwd(plan, q, k, v))
            torch.cuda.synchronize()
        wants.pop(-2)
        plan.close()
    long, side = torch.ones(1 << 28, device="cuda"), torch.cuda.Stream()

    def same(got, want):
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])

    for step in range(6):
        mask, want = masks[step % 3], wants[step % 3]
        first, out = ([torch.full_like(x, float("nan")) for x in want] for _ in range(2))
        plan, graph = dbsp.plan_sparse_attn(mask, block), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(4 * (step % 2)):
                long.mul_(1.0)
            dbsp.sparse_attn_fwd(plan, q, k, v, o=first[0], lse=first[1])
            graph.capture_begin()
            dbsp.sparse_attn_fwd(plan, q, k, v, o=out[0], lse=out[1])
            graph.capture_end()
        assert plan.run_order()["staged"]
        ticks, _ = plan.busy(side)
        assert np.array_equal(ticks > 0, plan.array(7) > 0)        # 7: blocks per partition
        same(first, want)
        for _ in range(3):
            out[0].zero_()
            out[1].zero_()
            graph.replay()
            same(out, want)
            same(dbsp.sparse_attn_fwd(plan, q, k, v), want)
        del graph
        plan.close()
        follower = dbsp.plan_sparse_attn(masks[(step + 1) % 3], block)
        same(dbsp.sparse_attn_fwd(follower, q, k, v), wants[(step + 1) % 3])
        follower.close()
