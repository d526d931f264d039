"""Plans on their way to the device, on the GPU: several streams, graph captures, plans given up while in use.

A plan of up to 64 KiB is fetched by a kernel in front of its first launch, a larger one copied on the
library's own stream; H picks either.  Results of a plan are bitwise the same from launch to launch.
"""

import numpy as np
import pytest
import torch

import paper_2511_23113_amd as dbsp

pytestmark = pytest.mark.gpu

SMALL, LARGE = 2, 96          # heads: about 12 KiB and 500 KiB of plan


def _case(H, seed=0, n=16):
    rng = np.random.default_rng(seed)
    mask = (rng.random((H, n, n)) < 0.4).astype(np.uint8)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    qkv = [torch.randn((1, H, n * 64, 64), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3)]
    return mask, qkv


def _plan(mask):
    return dbsp.plan_sparse_attn(mask, 64, num_partitions=64, mode=dbsp.MODE_ROUNDS, dynamic_tail=40)


def _expected(mask, qkv):
    plan = _plan(mask)
    o, lse = dbsp.sparse_attn_fwd(plan, *qkv)
    torch.cuda.synchronize()
    plan.close()
    return o, lse


def _same(got, want):
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("H", [SMALL, LARGE])
@pytest.mark.parametrize("eager_first", [True, False])
def test_captures_of_one_plan(H, eager_first):
    mask, qkv = _case(H)
    want = _expected(mask, qkv)
    plan = _plan(mask)
    if eager_first:
        _same(dbsp.sparse_attn_fwd(plan, *qkv), want)
    graphs = []
    for _ in range(2):                   # the second capture follows a launch that the first one recorded
        out = torch.empty_like(want[0]), torch.empty_like(want[1])
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            dbsp.sparse_attn_fwd(plan, *qkv, o=out[0], lse=out[1])
        graphs.append((g, out))
    for _ in range(3):
        for g, out in graphs:
            out[0].zero_()
            out[1].zero_()
            g.replay()
            _same(out, want)
        _same(dbsp.sparse_attn_fwd(plan, *qkv), want)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        got = dbsp.sparse_attn_fwd(plan, *qkv)
    _same(got, want)
    plan.close()


@pytest.mark.parametrize("H", [SMALL, LARGE])
def test_first_launch_waits_for_the_plan(H):
    """First launches while the copies to the device are kept busy, and second ones on another stream that is ordered
    behind the first on the device only, with a long kernel in front.  The plans' buffers held another mask's plan of
    the same shape before, so a launch that did not wait would work through that one."""
    cases = [_case(H, seed) for seed in (1, 2)]
    wants = [_expected(*c) for c in cases]
    host = torch.empty(1 << 27, dtype=torch.uint8, pin_memory=True)
    there = [torch.empty(1 << 27, dtype=torch.uint8, device="cuda") for _ in range(4)]
    long = torch.ones(1 << 28, device="cuda")
    side, others = torch.cuda.Stream(), [torch.cuda.Stream() for _ in there]
    torch.cuda.synchronize()
    for i in range(6):
        (mask, qkv), want = cases[i % 2], wants[i % 2]
        outs = [[torch.full_like(x, float("nan")) for x in want] for _ in range(2)]
        torch.cuda.synchronize()
        for x, st in zip(there, others):
            with torch.cuda.stream(st):
                x.copy_(host, non_blocking=True)
        plan = _plan(mask)
        if i >= 2:                       # (or nothing in front)
            long.mul_(1.0)
        dbsp.sparse_attn_fwd(plan, *qkv, o=outs[0][0], lse=outs[0][1])
        side.wait_stream(torch.cuda.current_stream())              # one plan's launches must not overlap
        with torch.cuda.stream(side):
            dbsp.sparse_attn_fwd(plan, *qkv, o=outs[1][0], lse=outs[1][1])
        for got in outs:
            _same(got, want)
        plan.close()


@pytest.mark.parametrize("H", [SMALL, LARGE])
def test_close_waits_for_the_last_launch(H):
    """Results may be read behind close() without any other synchronisation, here on a stream that waits for nothing."""
    mask, qkv = _case(H, 2, n=64)
    want = _expected(mask, qkv)
    plan, side = _plan(mask), torch.cuda.Stream()
    out = torch.full_like(want[0], float("nan")), torch.full_like(want[1], float("nan"))
    torch.cuda.synchronize()
    for _ in range(50):                  # the last launch ends milliseconds after the calls
        dbsp.sparse_attn_fwd(plan, *qkv, o=out[0], lse=out[1])
        out[0].fill_(float("nan"))
    dbsp.sparse_attn_fwd(plan, *qkv, o=out[0], lse=out[1])
    plan.close()
    with torch.cuda.stream(side):
        got = out[0].clone(), out[1].clone()
    side.synchronize()
    _same(got, want)


@pytest.mark.parametrize("H", [SMALL, LARGE])
def test_plans_dropped_while_in_use(H):
    """More plans than may wait for the GPU, each dropped right behind its launch, on two streams in turn;
    a buffer that went back too early would be overwritten by the next plan."""
    cases = [_case(H, seed) for seed in range(2)]
    wants = [_expected(*c) for c in cases]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got = []
    for i in range(24):
        mask, qkv = cases[i % 2]
        with torch.cuda.stream(side if i % 3 == 0 else torch.cuda.current_stream()):
            plan = _plan(mask)
            got.append(dbsp.sparse_attn_fwd(plan, *qkv))
            del plan
    torch.cuda.synchronize()
    for i, g in enumerate(got):
        _same(g, wants[i % 2])


def test_planning_inside_a_capture_beside_retired_plans():
    """Planning asks whether earlier plans' launches have ended: that must not spoil a capture."""
    mask, qkv = _case(SMALL, 3)
    want = _expected(mask, qkv)
    for _ in range(6):                    # the pools hold buffers from here on, and plans wait for the GPU
        plan = _plan(mask)
        dbsp.sparse_attn_fwd(plan, *qkv)
        del plan
    out = torch.empty_like(want[0]), torch.empty_like(want[1])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        kept = _plan(mask)
        dbsp.sparse_attn_fwd(kept, *qkv, o=out[0], lse=out[1])
    for _ in range(3):
        out[0].zero_()
        g.replay()
        _same(out, want)
        _same(dbsp.sparse_attn_fwd(kept, *qkv), want)
    kept.close()


@pytest.mark.parametrize("H", [SMALL, LARGE])
@pytest.mark.parametrize("close", [True, False])
def test_plans_given_up_inside_a_capture(H, close):
    """More plans than may wait for the GPU, launched just before a capture on another stream (some captured as well)
    and given up inside it: the capture stays whole, and no buffer goes back while its launch runs."""
    cases = [_case(H, seed, n=32) for seed in range(2)]
    wants = [_expected(*c) for c in cases]
    plans = [_plan(cases[i % 2][0]) for i in range(8)]
    spare = torch.empty_like(wants[0][0])
    torch.cuda.synchronize()
    got = []
    for i, plan in enumerate(plans):
        for _ in range(10):              # still running when the capture begins
            dbsp.sparse_attn_fwd(plan, *cases[i % 2][1], o=spare, want_lse=False)
        got.append(dbsp.sparse_attn_fwd(plan, *cases[i % 2][1]))
    out = torch.zeros_like(wants[0][0]), torch.zeros_like(wants[0][1])
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        graph.capture_begin()
        dbsp.sparse_attn_fwd(plans[0], *cases[0][1], o=spare, want_lse=False)
        out[0].add_(1.0)
        while plans:
            plan = plans.pop(0)
            if close:
                plan.close()
            del plan
        graph.capture_end()
    for i in range(8):                   # into the buffers that went back
        plan = _plan(cases[i % 2][0])
        got.append(dbsp.sparse_attn_fwd(plan, *cases[i % 2][1]))
    for i, g in enumerate(got):
        _same(g, wants[i % 2])
    assert not out[0].any()              # captured, not run


def test_an_earlier_error_leaves_no_buffers_in_use():
    """An error that the program left behind is reported by the call that fetches a plan; the plan can be used again, or
    dropped, and what follows in its buffers is right."""
    cases = [_case(SMALL, seed) for seed in range(2)]
    wants = [_expected(*c) for c in cases]
    hip = dbsp.load_library()                      # looks up the runtime it is linked to as well
    for i in range(4):
        (mask, qkv), want = cases[i % 2], wants[i % 2]
        out = torch.empty_like(want[0]), torch.empty_like(want[1])
        plan = _plan(mask)
        hip.hipSetDevice(1 << 20)                  # refused
        with pytest.raises(dbsp.DbspError):
            dbsp.sparse_attn_fwd(plan, *qkv, o=out[0], lse=out[1])
        if i < 2:
            dbsp.sparse_attn_fwd(plan, *qkv, o=out[0], lse=out[1])
            _same(out, want)
        del plan
        mask, qkv = cases[1 - i % 2]
        plan = _plan(mask)
        _same(dbsp.sparse_attn_fwd(plan, *qkv), wants[1 - i % 2])


@pytest.mark.parametrize("H", [SMALL, LARGE])
def test_a_graph_replayed_at_once_on_another_stream(H):
    """A graph holds nothing that waits for the plan's upload, so the plan has to be there when the capture ends, here
    with the copies to the device kept busy beside it."""
    mask, qkv = _case(H, 4)
    want = _expected(mask, qkv)
    out = torch.full_like(want[0], float("nan")), torch.full_like(want[1], float("nan"))
    host = torch.empty(1 << 28, dtype=torch.uint8, pin_memory=True)
    there = [torch.empty(1 << 28, dtype=torch.uint8, device="cuda") for _ in range(4)]
    side, others = torch.cuda.Stream(), [torch.cuda.Stream() for _ in there]
    torch.cuda.synchronize()
    for x, st in zip(there, others):
        with torch.cuda.stream(st):
            x.copy_(host, non_blocking=True)
    plan, graph = _plan(mask), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        graph.capture_begin()
        dbsp.sparse_attn_fwd(plan, *qkv, o=out[0], lse=out[1])
        graph.capture_end()
    for _ in range(2):
        graph.replay()                   # on the current stream
        _same(out, want)
        out[0].zero_()
        _same(dbsp.sparse_attn_fwd(plan, *qkv), want)
    plan.close()
