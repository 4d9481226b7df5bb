"""The work that users of this library have it do, as cases that can be timed and compared.

A case is one pass through the public entry points: a prefill (scores, thresholds and selection, attention), a
training step (the same and its whole backward), one decode step, a document in chunks (with or without the backward
of every chunk), or the importance scores alone.  `listed()` holds the ones to look at first, `draw()` gives more of
the same ranges.  Distributions are those of paper_2406_16747_amd/synth.py, drawn on the GPU: q, k, v ~ N(0,1)/sqrt(d),
scores ~ N(0,1) (what the timestep normalisation makes of any scorer), with a slow drift for training.
"""
import math

import torch

import paper_2406_16747_amd as spk

U_RING = 8192   # scores a decode state has in hand: a long generation, so that a state can be stepped thousands of times
QKV_RING = 8    # q, k, v of the coming decode steps, used in turn
DECODE_CTX = 4096   # tokens consumed before the first decode step (more than k + w everywhere)


def _prefill(B, H, n, d, k, w, Gu=1, gate_mode=0, dtype="bf16", hidden=0):
    return dict(kind="prefill", B=B, H=H, Gu=Gu, n=n, d=d, k=k, w=w, gate_mode=gate_mode, dtype=dtype, hidden=hidden)


def _train(B, H, n, d, k, w, Gu=1, gate_mode=0):
    return dict(kind="train", B=B, H=H, Gu=Gu, n=n, d=d, k=k, w=w, gate_mode=gate_mode, dtype="bf16")


def _decode(B, H, d, k, w, Gu=1, gate_mode=0):
    return dict(kind="decode", B=B, H=H, Gu=Gu, d=d, k=k, w=w, gate_mode=gate_mode, dtype="bf16")


def _chunks(B, H, chunk, count, d, k, w, Gu=1, gate_mode=0, train=False):
    return dict(kind="chunk_train" if train else "chunk_prefill", B=B, H=H, Gu=Gu, chunk=chunk, count=count, d=d, k=k,
                w=w, gate_mode=gate_mode, dtype="bf16")


def _scores(B, n, D, dtype="bf16"):
    return dict(kind="scores", B=B, n=n, D=D, dtype=dtype)


def listed():
    cases = {
        # one short fp32 head: the smallest call, a unit of development and of tests
        "prefill_one_head_fp32": _prefill(1, 1, 1024, 64, 64, 64, dtype="fp32"),
        # a GPT-2-small-shaped layer, the score network (768 features, normalised) included
        "prefill_gpt2_layer": _prefill(8, 12, 4096, 64, 256, 256, hidden=768),
        # a batch of prompts of a length nobody chose, k != w, gates on the values only
        "prefill_ragged": _prefill(2, 16, 5003, 128, 300, 200, gate_mode=1),
        # a Llama-7B-shaped layer over a long document
        "prefill_long": _prefill(1, 32, 32768, 128, 1024, 1024),
        # the same layer with a selection of its own for every head
        "prefill_per_head": _prefill(1, 32, 16384, 128, 1024, 1024, Gu=32),
        # training: forward and all gradients of a mid-size layer at 8 K tokens
        "train_layer": _train(4, 16, 8192, 128, 512, 512),
        # training of a GPT-2-small-shaped layer with the straight-through estimator, ragged length
        "train_gpt2_ste": _train(4, 12, 2000, 64, 128, 128, gate_mode=3),
        # one token for one user: latency
        "decode_one": _decode(1, 32, 128, 1024, 1024),
        # one token for each of 64 users: throughput of a serving batch
        "decode_batch": _decode(64, 32, 128, 1024, 1024),
        # a document of 32 K tokens in chunks of 8 K against the fixed-size cache
        "chunk_prefill": _chunks(1, 32, 8192, 4, 128, 1024, 1024),
        # training with chunk-wise recurrence
        "chunk_train": _chunks(1, 16, 4096, 4, 128, 512, 512, train=True),
        # importance scores of a Llama-7B-shaped hidden state
        "scores_llama": _scores(1, 32768, 4096),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(c):
    """Multiply-adds of the attention, near enough to bound a drawn case."""
    n = c.get("n") or c["chunk"] * c["count"]
    return c["B"] * c["H"] * n * min(n, c["k"] + c["w"]) * c["d"] * (3.5 if "train" in c["kind"] else 1.0)


MOST = 1.0 * 32 * 32768 * 2048 * 128   # the cost of prefill_long


def draw(rng):
    while True:
        kind = rng.choice(["prefill", "prefill", "prefill", "train", "train", "decode", "decode", "chunk_prefill",
                           "chunk_train", "scores"])
        if kind == "scores":
            n, D = _log(rng, 500, 32768), 8 * _log(rng, 64, 512)
            B = rng.randint(1, 8)
            if B * n * D <= 32768 * 4096:
                return _scores(B, n, D, rng.choice(["bf16", "bf16", "fp32"]))
            continue
        B, H, d = rng.choice([1, 1, 2, 3, 4, 8]), rng.choice([4, 8, 12, 16, 25, 32]), rng.choice([64, 128, 128])
        k, w = _log(rng, 64, 1024), _log(rng, 64, 1024)
        if rng.random() < 0.5:
            k = w = 64 * _log(rng, 1, 16)
        Gu = rng.choice([1, 1, 1, H])
        mode = rng.choice([0, 0, 0, 1, 2])
        if kind == "prefill":
            n = _log(rng, 500, 32768)
            if rng.random() < 0.15:   # fp32: development sizes
                c = _prefill(rng.randint(1, 2), rng.randint(1, 8), _log(rng, 500, 2048), rng.choice([32, 64, 128]),
                             min(k, 128), min(w, 128), 1, mode, "fp32")
            else:
                hidden = 64 * H if d == 64 and Gu == 1 else 0
                c = _prefill(B, H, n, d, k, w, Gu, mode, "bf16", hidden)
        elif kind == "train":
            c = _train(B, H, _log(rng, 500, 8192), d, k, w, Gu, rng.choice([0, 0, 1, 3]))
        elif kind == "decode":
            return _decode(rng.choice([1, 1, 2, 4, 8, 17, 32, 64]), H, d, k, w, Gu, mode)
        else:
            c = _chunks(min(B, 2), H, _log(rng, 512, 8192), rng.randint(2, 4), d, k, w, Gu,
                        rng.choice([0, 0, 1]), kind == "chunk_train")
        if _cost(c) <= MOST:
            return c


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def prepare(case, seed):
    g = _gen(seed)
    s = dict(case)
    dtype = torch.float32 if case["dtype"] == "fp32" else torch.bfloat16

    def normal(*shape, div=1.0, dt=None):
        t = torch.randn(*shape, device="cuda", generator=g, dtype=dt or dtype)
        return t.div_(div) if div != 1.0 else t

    if case["kind"] == "scores":
        s["x"] = normal(case["B"], case["n"], case["D"])
        s["wu"] = normal(case["D"], div=math.sqrt(case["D"]), dt=torch.float32)
        return s
    B, H, Gu, d = case["B"], case["H"], case["Gu"], case["d"]
    div = math.sqrt(d)
    if case["kind"] in ("prefill", "train"):
        n = case["n"]
        s["q"], s["k_"], s["v"] = (normal(B, H, n, d, div=div) for _ in range(3))
        if case.get("hidden"):
            s["x"] = normal(B, n, case["hidden"])
            s["wu"] = normal(case["hidden"], div=math.sqrt(case["hidden"]), dt=torch.float32)
        else:
            s["u"] = normal(B, Gu, n, dt=torch.float32)
        if case["kind"] == "train":
            s["u"] += 0.5 * torch.sin(torch.arange(n, device="cuda", dtype=torch.float32) / 256.0)
            s["dO"] = normal(B, H, n, d)
    elif case["kind"] == "decode":
        k, v = normal(B, H, DECODE_CTX, d, div=div), normal(B, H, DECODE_CTX, d, div=div)
        u = normal(B, Gu, DECODE_CTX, dt=torch.float32)
        tau, death = spk.sparsek_mask(u, case["k"])
        s["state"] = spk.DecodeState(B, H, Gu, d, case["k"], case["w"], dtype, case["gate_mode"], 1.0)
        spk.sparsek_decode_load(s["state"], k, v, u, tau, death)
        s["q"], s["k_"], s["v"] = ([normal(B, H, d, div=div) for _ in range(QKV_RING)] for _ in range(3))
        s["u"] = list(normal(U_RING, B, Gu, dt=torch.float32).unbind(0))
        s["step"] = 0
    else:
        c = case["chunk"]
        for name in ("q", "k_", "v"):
            s[name] = [normal(B, H, c, d, div=div) for _ in range(case["count"])]
        s["u"] = [normal(B, Gu, c, dt=torch.float32) for _ in range(case["count"])]
        if case["kind"] == "chunk_train":
            s["dO"] = [normal(B, H, c, d) for _ in range(case["count"])]
    return s


def _importance(s):
    return spk.sparsek_scores(s["x"], s["wu"], slope=2.0 ** -14, norm=True)


def run(s):
    kind = s["kind"]
    if kind == "scores":
        return _importance(s)
    if kind in ("prefill", "train"):
        u = _importance(s).unsqueeze(1) if s.get("hidden") else s["u"]
        k, w, mode = s["k"], s["w"], s["gate_mode"]
        tau, death = spk.sparsek_mask(u, k)
        o, lse = spk.sparsek_attn_fwd(s["q"], s["k_"], s["v"], u, tau, death, k, w, mode, 1.0)
        if kind == "prefill":
            return {"o": o, "lse": lse, "tau": tau, "death": death}
        dq, dk, dv, du = spk.sparsek_bwd(s["q"], s["k_"], s["v"], u, tau, death, o, lse, s["dO"], k, w, mode, 1.0)
        return {"o": o, "lse": lse, "tau": tau, "death": death, "dq": dq, "dk": dk, "dv": dv, "du": du}
    if kind == "decode":
        t = s["step"]
        s["step"] = t + 1
        i = t % QKV_RING
        return spk.sparsek_decode_step(s["state"], s["q"][i], s["k_"][i], s["v"][i], s["u"][t % U_RING])
    # a document: a fresh chunk state, then its chunks in order
    st = spk.ChunkState(s["B"], s["H"], s["Gu"], s["d"], s["k"], s["w"], spk.BF16, s["chunk"], s["gate_mode"], 1.0)
    out = []
    for i in range(s["count"]):
        q = s["q"][i]
        o = spk.sparsek_chunk_prefill(st, q, s["k_"][i], s["v"][i], s["u"][i])
        out.append([o, *spk.sparsek_chunk_bwd(st, q, o, s["dO"][i])] if kind == "chunk_train" else o)
    return out


def _pairs(n, k, w):
    """(query, key) pairs one head attends: query i its last min(i + 1, w) keys and min(k, i - w + 1) selected ones."""
    win = n * w - w * (w - 1) // 2 if n >= w else n * (n + 1) // 2
    m = max(n - w, 0)
    return win + (m * k - k * (k - 1) // 2 if m >= k else m * (m + 1) // 2)


def work(case):
    kind, B = case["kind"], case["B"]
    esz = 4 if case["dtype"] == "fp32" else 2
    if kind == "scores":
        n, D = case["n"], case["D"]
        return {"bytes": B * n * D * esz + D * 4 + B * n * 4, "flops": 2 * B * n * D}
    H, Gu, d, k, w = case["H"], case["Gu"], case["d"], case["k"], case["w"]
    if kind == "decode":
        slots = B * H * (k + w) * d
        return {"bytes": 2 * slots * esz + 4 * B * H * d * esz, "flops": 4 * slots}
    n = case["n"] if kind in ("prefill", "train") else case["chunk"] * case["count"]
    tensor, rows = B * H * n * d * esz, B * Gu * n * 4
    flops = 4 * d * _pairs(n, k, w) * B * H
    if kind == "prefill":
        hidden = B * n * case["hidden"] * esz
        return {"bytes": 4 * tensor + 4 * B * H * n + 3 * rows + hidden,
                "flops": flops + 2 * B * n * case["hidden"]}
    if kind == "train":   # two products forward, five backward
        return {"bytes": 8 * tensor + 4 * B * H * n + 4 * rows, "flops": 3.5 * flops}
    cache = 2 * B * H * (k + w) * d * esz * (case["count"] - 1)   # the retained rows, read once for every later chunk
    if kind == "chunk_prefill":
        return {"bytes": 4 * tensor + rows + cache, "flops": flops}
    return {"bytes": 8 * tensor + 2 * rows + cache, "flops": 3.5 * flops}


def tolerance(case):
    # fp32 storage: sums of up to a few thousand terms in another order; scores are summed in fp64 and rounded once.
    if case["dtype"] == "fp32" or case["kind"] == "scores":
        return {"rel": 1e-5, "max": 1e-3}
    # bf16 storage: outputs and the probabilities of the second product are rounded to 8 bits; lifetimes are whole
    # numbers and the same ("differ" 0).
    return {"rel": 1e-2, "max": 0.3}
