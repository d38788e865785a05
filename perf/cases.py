"""What the library is timed on: chunk attention (forward, backward, both; packed, split and hybrid chunks; head
dimensions 64, 96, 128 and 256) and the fused in-place cross-entropy, through the public entry points.

A case is a dict of plain values.  `op` is what one pass does:

  train    chunk_attn_fwd, then chunk_attn_bwd of the same chunk: what a pipeline stage does with a chunk
  static   chunk_attn_fwd_static: the forward that needs no workspace (tight loops, graph capture)
  chain    backward of two slices of one split sequence, the later slice first (it writes dK / dV, the earlier one adds to
           it), with float32 dK / dV buffers: how the gradients of a split sequence are carried
  ce       fused_ce_inplace on a buffer of logits that is refilled first (the operator overwrites its input)

and the chunk follows from `tail` and `context` (a slice of `tail` queries behind `context` keys; 0: none) and
from `tokens`, `median`, `sigma`, `low`, `high` (whole sequences packed behind it until they fill `tokens`, lengths log-normal and
clipped, drawn from `lengths_seed`; 0: none).  `lengths` names a fixed list of lengths instead.
"""
import math

import torch

import paper_2509_21275_amd as ca
import synth
from paper_2509_21275_amd.fused_ce import fused_ce_inplace

DEVICE = "cuda"
FIXED_LENGTHS = {"four_short": (256, 512, 128, 128)}


def _attn(name, op, heads, kv_heads, dim, tail=0, context=0, tokens=0, median=1024, sigma=1.0, low=128, high=4096,
          lengths_seed=0, lengths=""):
    return {"name": name, "op": op, "heads": heads, "kv_heads": kv_heads, "dim": dim, "tail": tail, "context": context,
            "tokens": tokens, "median": median, "sigma": sigma, "low": low, "high": high, "lengths_seed": lengths_seed,
            "lengths": lengths}


def _ce(name, rows, vocab, stride):
    return {"name": name, "op": "ce", "rows": rows, "vocab": vocab, "stride": stride}


def listed():
    return [
        # the smallest chunk of the workloads: four short sequences, bound by launches and latency
        _attn("packed_1k_d64", "train", 8, 8, 64, lengths="four_short"),
        # a small ragged hybrid chunk through the forward without a workspace, as a serving loop would call it
        _attn("static_ragged_d128", "static", 32, 8, 128, tail=203, context=1501, tokens=611, median=200, sigma=0.7, low=33,
              high=400, lengths_seed=3),
        # a fine slice of a long sequence: few queries, many keys
        _attn("slice_1k_of_32k", "train", 32, 8, 128, tail=1024, context=31744),
        # the last quarter of a 32K sequence
        _attn("split_32k_last_of_4", "train", 32, 8, 128, tail=8192, context=24576),
        # tail slice of a 64K sequence packed with short sequences
        _attn("hybrid_64k", "train", 32, 8, 128, tail=8192, context=57344, tokens=8192, median=1024, sigma=1.0, low=128, high=4096,
              lengths_seed=synth.BASE_SEED + 3),
        # skewed packed batch of 64K tokens
        _attn("packed_64k", "train", 32, 8, 128, tokens=65536, median=2048, sigma=1.2, low=128, high=16384,
              lengths_seed=synth.BASE_SEED + 4),
        # last slice of a 128K sequence with 64 query heads: the largest call
        _attn("split_128k_last_of_8", "train", 64, 8, 128, tail=16384, context=114688),
        # gradients carried across two odd slices of a split sequence in float32
        _attn("chain_f32_odd_slices", "chain", 32, 8, 128, tail=3193, context=4999),
        # the other head dimensions: 64 and 256 on the packed batch, 96 on the split one
        _attn("packed_64k_d64", "train", 32, 8, 64, tokens=65536, median=2048, sigma=1.2, low=128, high=16384,
              lengths_seed=synth.BASE_SEED + 4),
        _attn("split_32k_d96", "train", 32, 8, 96, tail=8192, context=24576),
        _attn("packed_64k_d256", "train", 32, 8, 256, tokens=65536, median=2048, sigma=1.2, low=128, high=16384,
              lengths_seed=synth.BASE_SEED + 4),
        # loss of one micro-batch at a vocabulary beyond 128K, rows as a padded projection leaves them
        _ce("ce_4k_x_152k", 4096, 151936, 152064),
    ]


def _log_uniform(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    """One more case of the same ranges.  Costs are kept under the largest listed case's by shortening."""
    op = rng.choices(["train", "static", "chain", "ce"], [12, 2, 2, 3])[0]
    if op == "ce":
        vocab = 8 * _log_uniform(rng, 1000, 32768)
        rows = max(1, min(_log_uniform(rng, 16, 16384), (1 << 30) // vocab))
        return {"op": "ce", "rows": rows, "vocab": vocab, "stride": vocab + 8 * rng.choice([0, 0, 1, 16])}
    heads, kv_heads = rng.choice([(32, 8), (32, 8), (64, 8), (8, 8), (8, 2)])
    dim = rng.choice([128, 128, 128, 128, 64, 96, 256])
    if op == "static":  # its scratch array is small: the layouts that fit it
        heads, kv_heads, dim = rng.choice([32, 8]), 8, rng.choice([64, 128])
    tail = context = tokens = 0
    if op == "static":
        tail, context, tokens = rng.randint(1, 400), rng.randint(0, 1500), rng.choice([0, rng.randint(64, 800)])
    elif op == "chain":
        tail, context = _log_uniform(rng, 100, 6000), _log_uniform(rng, 100, 6000)
    else:
        kind = rng.choice(["packed", "split", "hybrid"])
        if kind != "split":
            tokens = _log_uniform(rng, 500, 65536)
        if kind != "packed":
            tail, context = _log_uniform(rng, 100, 16384), _log_uniform(rng, 1, 65536)
            tokens = min(tokens, 16384)
    median = _log_uniform(rng, 150, 4096)
    case = _attn("", op, heads, kv_heads, dim, tail=tail, context=context, tokens=tokens, median=median,
                 sigma=rng.choice([0.5, 1.0, 1.2]), low=rng.choice([33, 128]), high=8 * median, lengths_seed=rng.randint(1, 1 << 30))
    if op == "static":
        case.update(median=150, sigma=0.7, low=33, high=400)
    while work(case)["flops"] > 1e14:
        case["context"] //= 2
    del case["name"]
    return case


def _segments(case):
    """[(q_start, q_len, kv_start, kv_len)] of the chunk, total query rows, total key rows."""
    segs, cq, ckv = [], 0, 0
    if case["tail"]:
        segs.append((0, case["tail"], 0, case["context"] + case["tail"]))
        cq, ckv = case["tail"], case["context"] + case["tail"]
    lens = FIXED_LENGTHS.get(case["lengths"], ())
    if case["tokens"]:
        lens = synth.lognormal_lengths(case["lengths_seed"], 0, case["tokens"], float(case["median"]), case["sigma"], case["low"],
                                       case["high"])
    for n in lens:
        segs.append((cq, n, ckv, n))
        cq += n
        ckv += n
    return segs, cq, ckv


def _pairs(segs):
    return sum(q * (kv - q) + q * (q + 1) // 2 for _, q, _, kv in segs)


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.bfloat16)

    if case["op"] == "ce":
        rows, vocab, stride = case["rows"], case["vocab"], case["stride"]
        projected = normal(rows, stride)[:, :vocab].mul_(2.0)
        targets = torch.randint(0, vocab, (rows,), generator=gen, device=DEVICE, dtype=torch.int32)
        targets[torch.rand(rows, generator=gen, device=DEVICE) < 0.05] = -100  # tokens that carry no loss
        return {"case": case, "projected": projected, "targets": targets, "loss": torch.empty(rows, device=DEVICE),
                "logits": torch.empty((rows, stride), dtype=torch.bfloat16, device=DEVICE)[:, :vocab], "scale": 1.0 / rows}

    H, Hk, d, scale = case["heads"], case["kv_heads"], case["dim"], case["dim"] ** -0.5
    if case["op"] == "chain":
        # one sequence of context + tail tokens cut into two slices: the later one sees every key
        total = case["context"] + case["tail"]
        k, v = normal(total, Hk, d), normal(total, Hk, d)
        slices = []
        for q_len, ctx in ((case["tail"], case["context"]), (case["context"], 0)):
            desc = ca.make_desc([(0, q_len, 0, ctx + q_len)], H, Hk, d, q_len, total, scale)
            q, do = normal(q_len, H, d), normal(q_len, H, d)
            ws = ca.alloc_workspace(desc, DEVICE)
            o, lse = torch.empty_like(q), torch.empty((H, q_len), device=DEVICE)
            ca.chunk_attn_fwd(desc, q, k, v, o, lse, ws)
            slices.append({"desc": desc, "q": q, "do": do, "o": o, "lse": lse, "ws": ws, "dq": torch.empty_like(q)})
        return {"case": case, "k": k, "v": v, "slices": slices, "dk": torch.empty(k.shape, device=DEVICE),
                "dv": torch.empty(v.shape, device=DEVICE)}

    segs, tq, tkv = _segments(case)
    desc = ca.make_desc(segs, H, Hk, d, tq, tkv, scale)
    q, k, v = normal(tq, H, d), normal(tkv, Hk, d), normal(tkv, Hk, d)
    state = {"case": case, "desc": desc, "q": q, "k": k, "v": v, "o": torch.empty_like(q),
             "lse": torch.empty((H, tq), device=DEVICE)}
    if case["op"] == "train":
        state.update(do=normal(tq, H, d), dq=torch.empty_like(q), dk=torch.empty_like(k), dv=torch.empty_like(v),
                     ws=ca.alloc_workspace(desc, DEVICE))
    return state


def run(state):
    op = state["case"]["op"]
    if op == "ce":
        state["logits"].copy_(state["projected"])  # stands for the projection that writes the logits
        fused_ce_inplace(state["logits"], state["targets"], state["loss"], state["scale"])
        return {"loss": state["loss"], "grad": state["logits"]}
    if op == "chain":
        for n, s in enumerate(state["slices"]):
            ca.chunk_attn_bwd_f32kv(s["desc"], s["q"], state["k"], state["v"], s["o"], s["do"], s["lse"], s["dq"], state["dk"],
                                    state["dv"], n > 0, s["ws"])
        return {"dq": [s["dq"] for s in state["slices"]], "dk": state["dk"], "dv": state["dv"]}
    if op == "static":
        ca.chunk_attn_fwd_static(state["desc"], state["q"], state["k"], state["v"], state["o"], state["lse"])
        return {"o": state["o"], "lse": state["lse"]}
    ca.chunk_attn_fwd(state["desc"], state["q"], state["k"], state["v"], state["o"], state["lse"], state["ws"])
    ca.chunk_attn_bwd(state["desc"], state["q"], state["k"], state["v"], state["o"], state["do"], state["lse"], state["dq"],
                      state["dk"], state["dv"], 0, state["ws"])
    return {n: state[n] for n in ("o", "lse", "dq", "dk", "dv")}


def work(case):
    if case["op"] == "ce":
        # the refill and the operator each read and write every logit once; two exponentials and a few operations per logit
        n = case["rows"] * case["vocab"]
        return {"bytes": 8 * n, "flops": 8 * n}
    H, Hk, d = case["heads"], case["kv_heads"], case["dim"]
    if case["op"] == "chain":
        total = case["context"] + case["tail"]
        pairs = total * (total + 1) // 2
        q_bytes, kv_bytes = 2 * total * H * d, 2 * total * Hk * d
        # reads q, o, dO, LSE, k, v (by both slices where both see it); writes dq; float32 dk / dv written, then added to
        return {"bytes": 4 * q_bytes + 4 * total * H + 2 * kv_bytes + 8 * total * Hk * d + 2 * 2 * 4 * case["context"] * Hk * d,
                "flops": 10 * d * pairs * H}
    segs, tq, tkv = _segments(case)
    pairs, q_bytes, kv_bytes = _pairs(segs), 2 * tq * H * d, 2 * tkv * Hk * d
    fwd = {"bytes": 2 * q_bytes + 2 * kv_bytes + 4 * tq * H, "flops": 4 * d * pairs * H}
    if case["op"] == "static":
        return fwd
    # backward: reads q, o, dO, LSE, k, v; writes dq, dk, dv
    return {"bytes": fwd["bytes"] + 4 * q_bytes + 4 * kv_bytes + 4 * tq * H, "flops": fwd["flops"] + 10 * d * pairs * H}


def tolerance(case):
    """Measured against the same mathematics in 64 bits on the same bf16 inputs, at chunks of a few thousand rows of every head
    dimension (rel: 2-norm; max: largest difference over the larger of value and root mean square):
    O 1.9e-3 .. 2.4e-3 and 2.2e-2, dQ / dK / dV 2.3e-3 .. 3.0e-3 and 8.8e-2 (P and dS are rounded to bf16 before their
    products, the results once more); stated are four times that.  Gradients of the logits are one bf16 rounding, 2^-9
    of the value at most (measured 3.4e-3 of it once the row's log-sum-exp is in 32 bits)."""
    if case["op"] == "ce":
        return {"rel": 4e-3, "max": 1.6e-2}
    if case["op"] == "static":
        return {"rel": 1e-2, "max": 0.09}
    return {"rel": 1.2e-2, "max": 0.35}
