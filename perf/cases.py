"""The work a training run gives this library, as cases that can be timed and checked.

Two entry points carry it: the outer step (subgroups drawn by `plan_groups`, then `outer_step` over
the whole arena) and the replica-spread pass that monitors it. A case names one call by its layout,
number of replicas, subgroup size and storage types; `run` makes that call the way a training
program does, with the launch plan and the arena it keeps between outer steps.

Arena sizes are those of `workloads/` (GPT-style blocks of 768/12/3072, 2048/24/8192, 4096/32/16384;
4096 ragged tensors in 124 439 808 elements; the flat 2^20 arena; the small ragged test arena), with
as many replicas as leave room for several arenas on one GPU.
"""
import math

import numpy as np
import torch

import paper_2506_10911_amd as nl

ALIGN_ELEMS = 64                # worker rows start at multiples of this many elements
HPARAMS = (0.9, 0.7, 1.0)       # outer momentum, outer learning rate, pull towards the subgroup mean
INIT_STD = 0.02                 # slow weights
APART_STD = 5e-4                # how far the replicas' slow weights have drifted apart
MOMENTUM_STD = 1e-3             # outer momentum after a few outer steps
DRIFT_STD = 1e-3                # what an inner phase does to the fast weights
SEED = 17                       # of the run's subgroup plan
MOST_BYTES = 58_012_729_344     # the largest listed case: stage1p3b, W = 8, float fast weights
LEAST_BYTES = 1 << 21


def _step(name, layout, W, n, theta, present=0, **sizes):
    return dict(name=name, op="step", layout=layout, W=W, n=n, theta=theta, present=present or W, **sizes)


def _spread(name, layout, W, x, static_scratch=False, **sizes):
    return dict(name=name, op="spread", layout=layout, W=W, x=x, static_scratch=static_scratch, **sizes)


def listed():
    return [
        # A unit-test or toy model: the call itself (host work, one short launch) is most of the time.
        _step("small_gapped_w8_n4_bf16", "gapped", 8, 4, "bf16", tensors=24, total=87_000),
        # The flat 2^20-element arena of the benchmark's smallest configuration.
        _step("tiny_w4_pairs_f32", "flat", 4, 2, "f32", total=1 << 20),
        # One 768-wide block, eight replicas of which one has dropped out of this round: the seven that
        # answered form two pairs and a triple.
        _step("block768_w8_dropout_bf16", "gpt", 8, 2, "bf16", present=7, d=768, f=3072, blocks=1, vocab=0),
        # Many small odd tensors with unowned elements between them (adapters, norms, biases).
        _step("adapters_gapped_w8_pairs_f32", "gapped", 8, 2, "f32", tensors=1024, total=4_000_000),
        # A subgroup size that is no power of two.
        _step("block2048_w12_n3_bf16", "gpt", 12, 3, "bf16", d=2048, f=8192, blocks=1, vocab=0),
        # The 125M model on eight replicas in random pairs: the paper's smallest training run.
        _step("gpt125m_w8_pairs_f32", "gpt", 8, 2, "f32", d=768, f=3072, blocks=12, vocab=50257),
        # The same model on sixteen replicas with all of them in one group (DiLoCo's outer step).
        _step("gpt125m_w16_diloco_bf16", "gpt", 16, 16, "bf16", d=768, f=3072, blocks=12, vocab=50257),
        # 4096 ragged tensors with gaps, subgroups of four.
        _step("ragged_gapped_w16_n4_f32", "gapped", 16, 4, "f32", tensors=4096, total=124_439_808),
        # One pipeline stage of the 1.3B model on eight replicas in pairs: the largest.
        _step("stage1p3b_w8_pairs_f32", "gpt", 8, 2, "f32", d=2048, f=8192, blocks=6, vocab=0),
        # Replica spread of the slow weights of the 125M model, as it is logged beside the loss.
        _spread("spread_gpt125m_w8_f32", "gpt", 8, "f32", d=768, f=3072, blocks=12, vocab=50257),
        # Replica spread of the bf16 fast weights of one 4096-wide block over sixteen replicas.
        _spread("spread_block4096_w16_bf16", "gpt", 16, "bf16", d=4096, f=16384, blocks=1, vocab=0),
        # Replica spread of a small ragged arena over a number of replicas that is no power of two, through
        # the entry point that allocates nothing.
        _spread("spread_adapters_w12_f32", "gapped", 12, "f32", static_scratch=True, tensors=1024, total=4_000_000),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    W = rng.choice([2, 3, 4, 5, 6, 7, 8, 8, 8, 10, 12, 15, 16, 16, 16, 24, 32, 48, 64])
    stored = rng.choice(["f32", "bf16"])
    layout = rng.choice(["gpt", "gpt", "gapped", "gapped", "tight", "flat"])
    step = rng.random() < 0.7
    per_element = W * ((24 if stored == "f32" else 20) if step else (4 if stored == "f32" else 2))
    total = int(_log_uniform(rng, LEAST_BYTES, 0.9 * MOST_BYTES * (1.0 if step else 0.25)) / per_element)
    total = min(max(total, 4097), 1_700_000_000)
    if layout == "gpt":
        blocks = rng.randint(1, 12)
        d = max(int(math.sqrt(total / (12 * blocks))), 8)
        sizes = dict(d=d, f=4 * d, blocks=blocks, vocab=0)
    elif layout == "flat":
        sizes = dict(total=total)
    else:
        sizes = dict(tensors=int(_log_uniform(rng, 8, min(4096, max(9, total // 128)))), total=total)
    if not step:
        return dict(op="spread", layout=layout, W=W, x=stored, static_scratch=rng.random() < 0.3, **sizes)
    fits = [n for n in range(1, W + 1) if W % n == 0]
    n = 2 if W % 2 == 0 and rng.random() < 0.5 else rng.choice(fits)
    present = W - 1 if rng.random() < 0.2 and n < W else W
    return dict(op="step", layout=layout, W=W, n=n, theta=stored, present=present, **sizes)


def _tensors(case):
    """Sizes of the arena's tensors, in order."""
    layout = case["layout"]
    if layout == "flat":
        return [case["total"]]
    if layout == "gpt":
        d, f = case["d"], case["f"]
        block = [d, d, 3 * d * d, 3 * d, d * d, d, d, d, d * f, f, f * d, d]
        if case["vocab"]:
            return [case["vocab"] * d, 1024 * d] + case["blocks"] * block + [d, d]
        return case["blocks"] * block
    # Odd sizes, log-uniform over 14 binary orders of magnitude, scaled to the arena's total.
    rng = np.random.default_rng([4, 0x7261, case["tensors"]])
    s = np.floor(2.0 ** rng.uniform(6.0, 20.0, size=case["tensors"]))
    s = np.maximum(np.floor(s * (case["total"] / s.sum())), 64).astype(np.int64) | 1
    return [int(v) for v in s]


def _segments(case):
    """(offset, numel) of every tensor in a worker's row, and the row's length."""
    sizes = _tensors(case)
    gaps = [0] * len(sizes)
    if case["layout"] == "gapped":      # 1..7 elements that belong to nobody after every tensor
        gaps = np.random.default_rng([4, 0x6170]).integers(1, 8, size=len(sizes)).tolist()
    segments, at = [], 0
    for size, gap in zip(sizes, gaps):
        segments.append((at, size))
        at += size + gap
    return segments, -(-at // ALIGN_ELEMS) * ALIGN_ELEMS


def _rows(case, seed, stride, want):
    """The arrays named in `want`, [W, stride] each: slow weights around a common point, momentum, and
    fast weights an inner phase away from the slow ones."""
    W, dev = case["W"], "cuda"
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    base = torch.empty(stride, device=dev).normal_(0.0, INIT_STD, generator=gen)
    out = {}
    if "phi" in want:
        out["phi"] = torch.empty((W, stride), device=dev)
    if "delta" in want:
        out["delta"] = torch.empty((W, stride), device=dev).normal_(0.0, MOMENTUM_STD, generator=gen)
    stored = case.get("theta", case.get("x"))
    if "theta" in want:
        out["theta"] = torch.empty((W, stride), device=dev, dtype=torch.bfloat16 if stored == "bf16" else torch.float32)
    row = torch.empty(stride, device=dev)
    for w in range(W):
        row.normal_(0.0, APART_STD, generator=gen).add_(base)
        if "phi" in want:
            out["phi"][w].copy_(row)
        if "theta" in want:
            out["theta"][w].copy_(torch.empty(stride, device=dev).normal_(0.0, DRIFT_STD, generator=gen).add_(row))
    return out


def _alive(case):
    """The workers of this round, and the positions and offsets of their groups are drawn over them:
    the worker in the middle is the one that dropped out."""
    return np.array([w for w in range(case["W"]) if case["present"] == case["W"] or w != case["W"] // 2], dtype=np.int32)


def _arrays(case, seed):
    segments, stride = _segments(case)
    if case["op"] == "step":
        return segments, stride, _rows(case, seed, stride, ("phi", "delta", "theta"))
    name = "phi" if case["x"] == "f32" else "theta"
    return segments, stride, {"x": _rows(case, seed, stride, (name,))[name]}


def prepare(case, seed):
    segments, stride, arrays = _arrays(case, seed)
    state = dict(case=case, arrays=arrays, step=0)
    W = case["W"]
    if case["op"] == "step":
        state["alive"] = _alive(case)
        state["plan"] = nl.LaunchPlan(arrays["phi"], arrays["delta"], arrays["theta"], stride, W,
                                      nl.BF16 if case["theta"] == "bf16" else nl.F32, segments)
    else:
        x = arrays["x"]                 # a plan depends on the layout alone
        state["plan"] = nl.LaunchPlan(x, x, x, stride, W, nl.BF16 if case["x"] == "bf16" else nl.F32, segments)
        state["out"] = torch.zeros(len(segments) + 1, dtype=torch.float64, device="cuda")
    return state


def _groups(case, step, alive):
    """The round's subgroups: the library's plan over the workers that answered; what is left over when
    their number is no multiple of n joins the last group."""
    present, n = case["present"], case["n"]
    if present == case["W"]:
        return nl.plan_groups(SEED, step, present, n)
    whole = present - present % n
    members, offsets = nl.plan_groups(SEED, step, whole, n)
    members = alive[np.concatenate([members, np.arange(whole, present, dtype=np.int32)])]
    offsets[-1] = present
    return members, offsets


def run(state):
    case, arrays = state["case"], state["arrays"]
    if case["op"] == "step":
        members, offsets = _groups(case, state["step"], state["alive"])
        nl.outer_step(state["plan"], arrays["phi"], arrays["delta"], arrays["theta"], HPARAMS, members, offsets)
        state["step"] += 1
        return {"phi": arrays["phi"], "delta": arrays["delta"], "theta": arrays["theta"]}
    spread = nl.replica_spread_noalloc if case["static_scratch"] else nl.replica_spread
    spread(state["plan"], arrays["x"], nl.BF16 if case["x"] == "bf16" else nl.F32, state["out"])
    return state["out"]


def work(case):
    segments, _ = _segments(case)
    elements = sum(numel for _, numel in segments)
    if case["op"] == "step":
        # phi, delta and theta of every worker in the round read and written once
        updates = elements * case["present"]
        return {"bytes": updates * (24 if case["theta"] == "f32" else 20), "flops": updates * 11}
    return {"bytes": elements * case["W"] * (4 if case["x"] == "f32" else 2) + 8 * (len(segments) + 1),
            "flops": elements * case["W"] * 4}


def tolerance(case):
    if case["op"] == "step":
        # The sums over a subgroup in another order move the momentum by a few roundings of the slow weights.
        # A bf16 fast weight that sits on a tie may then fall to the other side: one unit in its last place.
        return {"rel": 5e-6, "max": 2e-4} if case["theta"] == "f32" else {"rel": 5e-5, "max": 1e-2}
    # float sums over the replicas of one element in another order; pooled in double
    return {"rel": 2e-7}


def exact(case, seed):
    segments, stride, arrays = _arrays(case, seed)
    if case["op"] == "spread":
        return _exact_spread(segments, arrays["x"])
    out = {k: torch.empty(v.shape, dtype=torch.float64, device=v.device) for k, v in arrays.items()}
    for k, v in arrays.items():
        out[k].copy_(v)
    del arrays
    owned = torch.zeros(stride, dtype=torch.bool, device="cuda")
    for offset, numel in segments:
        owned[offset:offset + numel] = True
    members, offsets = _groups(case, 0, _alive(case))
    alpha, beta, gamma = (float(np.float32(h)) for h in HPARAMS)
    chunk = 1 << 25
    for lo, hi in zip(offsets[:-1].tolist(), offsets[1:].tolist()):
        rows = torch.from_numpy(members[lo:hi].astype(np.int64)).cuda()
        for a in range(0, stride, chunk):
            b = min(a + chunk, stride)
            mine = owned[a:b]
            mean_phi = torch.zeros(b - a, dtype=torch.float64, device="cuda")
            mean_theta = torch.zeros_like(mean_phi)
            for w in rows.tolist():
                mean_phi += out["phi"][w, a:b]
                mean_theta += out["theta"][w, a:b]
            mean_phi /= hi - lo
            mean_theta /= hi - lo
            for w in rows.tolist():
                phi, delta, theta = (out[k][w, a:b] for k in ("phi", "delta", "theta"))
                d = alpha * delta - beta * (mean_phi - mean_theta) - gamma * (phi - mean_phi)
                delta.copy_(torch.where(mine, d, delta))
                phi.copy_(torch.where(mine, phi + d, phi))
                theta.copy_(torch.where(mine, phi, theta))
    return out


def _exact_spread(segments, x):
    W, stride = x.shape
    variance = torch.empty(stride, dtype=torch.float64, device=x.device)
    chunk = 1 << 24
    for a in range(0, stride, chunk):
        b = min(a + chunk, stride)
        mean = torch.zeros(b - a, dtype=torch.float64, device=x.device)
        for w in range(W):
            mean += x[w, a:b]
        mean /= W
        v = torch.zeros_like(mean)
        for w in range(W):
            v += (x[w, a:b].double() - mean).square_()
        variance[a:b] = v / W
    sums = torch.stack([variance[o:o + n].sum() for o, n in segments])
    counts = torch.tensor([n for _, n in segments], dtype=torch.float64, device=x.device)
    return torch.cat([(sums / counts).sqrt(), (sums.sum() / counts.sum()).sqrt().reshape(1)])
