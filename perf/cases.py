"""Cases by which the speed of block-sparse attention is measured, over the range a video-DiT program uses.

A case is a dict of plain values.  Attention cases: B, H, nQ, nK (mask blocks), block, d; `pattern` and
`spread` / `lo` / `hi` (the heads' densities) say what the masks look like; `plan` says how the program
holds its plans: "each" (a mask from the step's own activations: planned on every call), "carried" (the
same, with the placement carried over from the previous step's plan), "kept" (masks settled offline:
planned once per layer).  Partition cases: the host-side division of a mask among the GPUs of a ring.
"""

import numpy as np
import torch

import paper_2511_23113_amd as dbsp

REUSE_THRESHOLD = 1.10        # the paper's P_s
PLACEMENTS = {
    "greedy": {},                                                                        # plan_sparse_attn's defaults
    "rounds": dict(mode=dbsp.MODE_ROUNDS, locality_groups=8, dynamic_tail=40),           # what bench.py runs
}


def attention(name, H, nQ, nK, block, d, pattern, spread, lo, hi, plan, placement, B=1, pair="no", lse=True):
    return dict(name=name, kind="attention", B=B, H=H, nQ=nQ, nK=nK, block=block, d=d, pattern=pattern, spread=spread, lo=lo, hi=hi,
                plan=plan, placement=placement, pair=pair, lse=lse)


def listed():
    return [
        # the smallest call: 512 tokens, two heads, a new mask on every call (latency, launches, host work)
        attention("tiny_step", 2, 8, 8, 64, 64, "diagonal", "linear", 0.25, 0.55, "each", "greedy"),
        # a short clip at low resolution with offline masks: one launch per call, an odd grid, Nq != Nk
        attention("short_clip_kept", 12, 21, 23, 128, 128, "diagonal", "linear", 0.30, 0.80, "kept", "greedy"),
        # CogVideoX-5B-like layer (275 blocks of 64 tokens, d = 64), masks from the step's own scores
        attention("cogvideo_step", 48, 275, 275, 64, 64, "band_sink", "linear", 0.05, 0.45, "each", "rounds"),
        # Wan-14B-like layer at 480p, the benchmark's workload: dynamic masks with a 3D window and clusters
        attention("wan_step", 40, 256, 256, 128, 128, "window_clusters", "linear", 0.05, 0.60, "each", "rounds"),
        # HunyuanVideo-like layer at 720p: the largest masks and tensors, heads either sparse or half dense
        attention("hunyuan_step", 24, 928, 928, 128, 128, "frames", "bimodal", 0.05, 0.50, "each", "rounds"),
        # one device's share of a layer under head and block split; denoising steps carry the placement over
        attention("share_carried", 10, 128, 256, 128, 128, "diagonal", "geometric", 0.04, 0.55, "carried", "rounds"),
        # 64-token masks settled offline after token reordering (neighbouring rows alike) at d = 128
        attention("reordered64_kept", 40, 512, 512, 64, 128, "clusters", "linear", 0.05, 0.50, "kept", "rounds", pair="auto"),
        # 64-token dynamic masks without such structure at d = 128, an odd number of blocks
        attention("scattered64_step", 24, 301, 301, 64, 128, "diagonal", "linear", 0.08, 0.40, "each", "rounds", pair="auto"),
        # a d = 64 layer with 128-token blocks, guided sampling (conditional and unconditional batch entry), defaults
        attention("guided_d64_kept", 30, 137, 137, 128, 64, "frames", "linear", 0.10, 0.50, "kept", "greedy", B=2),
        # the first denoising steps, which sparse-attention methods leave dense
        attention("dense_steps_kept", 10, 97, 97, 128, 128, "diagonal", "linear", 1.0, 1.0, "kept", "rounds"),
        # a long sequence at very low density: short rows, few of them sharing a KV block; LSE not wanted
        attention("long_sparse_step", 16, 513, 513, 128, 128, "window_clusters", "geometric", 0.02, 0.08, "each", "rounds", lse=False),
        # dual-balanced planning for eight GPUs: heads over a Ulysses group, blocks over a ring, on the host
        dict(name="ring_plan", kind="partition", H=40, nQ=256, nK=256, ranks=8, reward=1.0,
             pattern="window_clusters", spread="linear", lo=0.05, hi=0.60),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more case of the same ranges; at most a quarter of the largest listed case's operations."""
    cap = max(work(c)["flops"] for c in listed()) / 4
    pattern = rng.choice(["diagonal", "band_sink", "window_clusters", "frames", "clusters"])
    spread = rng.choice(["linear", "geometric", "bimodal"])
    lo = round(0.02 * 10 ** rng.random(), 4)
    hi = round(min(1.0, lo * (2 + 6 * rng.random())), 4)
    if rng.random() < 1 / 12:
        n = _log_int(rng, 64, 700)
        return dict(kind="partition", H=_log_int(rng, 8, 48), nQ=n, nK=n, ranks=rng.choice([2, 4, 8]), reward=rng.choice([0.0, 0.05, 1.0]),
                    pattern=pattern, spread=spread, lo=lo, hi=hi)
    while True:
        block, d = rng.choice([64, 128]), rng.choice([64, 128])
        H = _log_int(rng, 2, 48)
        nQ = _log_int(rng, 6, 900)
        nK = nQ if rng.random() < 0.7 else _log_int(rng, max(6, nQ // 2), 2 * nQ)
        case = attention(None, H, nQ, nK, block, d, pattern, spread, lo, hi, rng.choice(["each", "each", "carried", "kept"]),
                         rng.choice(["greedy", "rounds"]), B=rng.choice([1, 1, 1, 2]),
                         pair="auto" if block == 64 and d == 128 else "no", lse=rng.random() < 0.8)
        del case["name"]
        if work(case)["flops"] <= cap and case["B"] * H * max(nQ, nK) * block * d <= 3 << 27 and H * nQ * nK <= 20 << 20:
            return case


def _counts(case):
    """Active blocks of every head, lightest first: fixed by the case; the seed says which head gets which."""
    H, lo, hi = case["H"], case["lo"], case["hi"]
    x = (np.arange(H) + 0.5) / H
    if case["spread"] == "linear":
        dens = lo + (hi - lo) * x
    elif case["spread"] == "geometric":
        dens = lo * (hi / lo) ** x
    else:                                        # half the heads near lo (up to twice), half near hi (from 0.6 of it)
        dens = np.where(x < 0.5, lo * (1 + 2 * x), hi * (0.6 + 0.8 * (x - 0.5)))
    n = case["nQ"] * case["nK"]
    return np.clip(np.rint(np.minimum(dens, 1.0) * n), 1, n).astype(np.int64)


def _scores(case, gen):
    """One score per block of one head: the head's mask is its highest-scored blocks."""
    nQ, nK, pattern = case["nQ"], case["nK"], case["pattern"]
    s = torch.rand((nQ, nK), generator=gen, device="cuda")
    I, J = torch.arange(nQ, device="cuda")[:, None], torch.arange(nK, device="cuda")[None, :]
    I = I * nK // nQ                             # the diagonal of a rectangular grid
    if "clusters" in pattern:                    # whole 4 x 4 groups of blocks, from a random offset, in random order
        a, b = torch.randint(0, 4, (2,), generator=gen, device="cuda").tolist()
        group = torch.rand(((nQ + 7) // 4, (nK + 7) // 4), generator=gen, device="cuda")
        s = s * 1e-6 + group.repeat_interleave(4, 0).repeat_interleave(4, 1)[a:a + nQ, b:b + nK]
    if pattern == "diagonal":
        first = I == J
    elif pattern == "band_sink":
        first = ((I - J).abs() <= 1) | (J < 2)
    elif pattern == "window_clusters":
        cols = torch.zeros((1, nK), dtype=torch.bool, device="cuda")
        cols[0, torch.randint(0, nK, (4,), generator=gen, device="cuda")] = True
        first = cols | ((I - J).abs() <= 1) | ((I - J - 16).abs() <= 1) | ((I - J + 16).abs() <= 1)
    elif pattern == "frames":
        first = ((I - J).abs() <= 2) | (I // 32 == J // 32)
    else:
        first = (I < 0) & (J < 0)
    return s + 2.0 * first


def _masks(case, gen, steps=1):
    """`steps` masks uint8 [H, nQ, nK] of consecutive denoising steps, a fifth of the blocks drawn anew at each."""
    counts = torch.from_numpy(_counts(case)).cuda()[torch.randperm(case["H"], generator=gen, device="cuda")].tolist()
    masks = [torch.zeros((case["H"], case["nQ"] * case["nK"]), dtype=torch.uint8, device="cuda") for _ in range(steps)]
    for h, count in enumerate(counts):
        s = _scores(case, gen)
        for m in masks:
            m[h, torch.sort(s.reshape(-1), descending=True, stable=True).indices[:count]] = 1
            if steps > 1:
                again = torch.rand(s.shape, generator=gen, device="cuda") < 0.2
                s = torch.where(again & (s < 2.0), torch.rand(s.shape, generator=gen, device="cuda"), s)
    return [m.reshape(case["H"], case["nQ"], case["nK"]).cpu().numpy() for m in masks]


def _plan_options(case):
    return dict(PLACEMENTS[case["placement"]], max_batch=case["B"])


def _plan(case, mask):
    return dbsp.plan_sparse_attn(mask, case["block"], head_dim=case["d"], pair_rows="auto" if case["pair"] == "auto" else False,
                                 **_plan_options(case))


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    masks = _masks(case, gen, 2 if case.get("plan") == "carried" else 1)
    if case["kind"] == "partition":
        return dict(case=case, mask=masks[0], blocks_per_head=masks[0].sum(axis=(1, 2), dtype=np.int64))

    def tensor(n):
        shape = (case["B"], case["H"], n * case["block"], case["d"])
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)
    state = dict(case=case, mask=masks[-1], q=tensor(case["nQ"]), k=tensor(case["nK"]), v=tensor(case["nK"]), plan=None)
    if case["plan"] == "kept":
        state["plan"] = _plan(case, masks[0])
    elif case["plan"] == "carried":
        state["previous"] = _plan(case, masks[0])
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "partition":
        heads = dbsp.partition_heads(state["blocks_per_head"], case["ranks"])
        blocks = dbsp.partition_blocks(state["mask"], case["ranks"], reward=case["reward"])
        return {"gpu_of_head": np.asarray(heads["gpu_of_head"]), "loads": np.asarray(heads["loads"]), "rho_heads": heads["rho"],
                "gpu_of_q": np.asarray(blocks["gpu_of_q"]), "chunk_of_kv": np.asarray(blocks["chunk_of_kv"]),
                "work": np.asarray(blocks["work"]), "rho_blocks": blocks["rho"], "moved": np.asarray([blocks["moved_q"], blocks["moved_kv"]])}
    if case["plan"] == "each":          # the layer keeps its plan until the next step's takes its place
        state["plan"] = _plan(case, state["mask"])
    elif case["plan"] == "carried":
        state["plan"], _, _ = dbsp.plan_sparse_attn_reuse(state["previous"], state["mask"], REUSE_THRESHOLD, **_plan_options(case))
    o, lse = dbsp.sparse_attn_fwd(state["plan"], state["q"], state["k"], state["v"], want_lse=case["lse"])
    return {"o": o, "lse": lse} if case["lse"] else {"o": o}


def work(case):
    pairs = int(_counts(case).sum())
    mask_bytes = case["H"] * case["nQ"] * case["nK"]
    if case["kind"] == "partition":
        return {"bytes": mask_bytes + 4 * (case["H"] + case["nQ"] + case["nK"]) + 8 * case["ranks"] ** 2, "flops": 0}
    rows, keys = case["B"] * case["H"] * case["nQ"] * case["block"], case["B"] * case["H"] * case["nK"] * case["block"]
    moved = 2 * case["d"] * (2 * rows + 2 * keys) + (4 * rows if case["lse"] else 0) + (0 if case["plan"] == "kept" else mask_bytes)
    return {"bytes": moved, "flops": 4 * case["block"] ** 2 * case["d"] * pairs * case["B"]}


def tolerance(case):
    # bf16 inputs, probabilities and outputs with f32 sums; plans are integers
    return "exact" if case["kind"] == "partition" else {"rel": 1e-2, "max": 0.1}
