"""The work that a user of this library has it do, as cases that can be timed and compared.

Three kinds of pass, all through the binding's own calls:

  request  one mesh from start to end: the condition memory of every sequence, a given first block of tokens (a mesh that
           is continued), and fm_generate to a number of faces.
  step     one decode step of a mesh under way: fm_draft, fm_verify_block, fm_commit with a full sliding window of K/V
           behind it.  Passes follow each other along the stream; the window keeps their cost the same.
  admit    new sequences enter: fm_prefill_condition of each, then the first block through fm_verify_block.

Models are random like the repository's benchmark models, with one difference: row pi(t) of the output head is the
embedding of token t (pi one cycle through the coordinate bins) and embeddings are four times as large.  The backbone then predicts
pi(t) after t with the clear margin that a trained model has and a random one lacks: streams do not hang on rounding, and the
continuation is known without decoding it, so that drafts can be right as often as the paper's are (replay, p = 0.93).
Every block, head and cache is computed in full all the same.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2511_15618_amd import FlashMesh, FmConfig

KEEP = 0.93            # share of draft tokens that are right: mean accepted lengths of the paper's 9-9 model
STREAM_FACES = 40000   # length of the streams that `step` passes walk along


def _case(name, kind, d, heads, c, v, f, *, bins=1024, mem=4096, dtype="bf16", batch=1, dc=2, m=9, n=9, faces=0, capacity=0,
          window=0, temperature=0.0, correct=0, speculative=True):
    return {"name": name, "kind": kind, "d": d, "heads": heads, "c": c, "v": v, "f": f, "bins": bins, "mem": mem, "dtype": dtype,
            "batch": batch, "dc": dc, "m": m, "n": n, "faces": faces, "capacity": capacity, "window": window,
            "temperature": temperature, "correct": correct, "speculative": speculative}


def listed():
    return [
        # the benchmark's smallest configuration, whole: 10 faces in fp32, three coordinate heads
        _case("request_tiny_f32", "request", 256, 4, 4, 4, 4, bins=128, mem=256, dtype="f32", dc=3, m=0, n=0, faces=10, capacity=10),
        # a mesh under way on the small model (500 faces of context): the shortest step, all latency
        _case("step_small_b1", "step", 512, 8, 4, 8, 8, mem=2048, window=4500),
        # the headline: one sequence on the medium model at half of its 18000-token context
        _case("step_medium_b1", "step", 1024, 16, 8, 16, 16, window=9000),
        # the batched headline: eight sequences with accepted lengths of their own
        _case("step_medium_b8", "step", 1024, 16, 8, 16, 16, batch=8, window=4500),
        # the large model, blocks of two faces
        _case("step_large_b4", "step", 1536, 24, 8, 16, 24, batch=4, m=15, n=18, window=4500),
        # the paper's widest model: 16 heads of 128, 18-15 drafts
        _case("step_d2048_hd128_b1", "step", 2048, 16, 4, 8, 12, m=15, n=18, window=3600),
        # a few users at once, odd batch, heads of 96
        _case("step_d768_hd96_b3", "step", 768, 8, 4, 8, 12, mem=1369, batch=3, window=2700),
        # first faces of a mesh on the medium model: condition memory, short context
        _case("request_medium_b1", "request", 1024, 16, 8, 16, 16, faces=24, capacity=2000),
        # plain one-token decoding of the small model (no draft heads), what speculation is compared with
        _case("request_small_plain", "request", 512, 8, 4, 8, 8, mem=2048, faces=8, capacity=500, speculative=False),
        # sampled decoding with the correct stage, five sequences, ragged memory, 18-token blocks
        _case("request_sampled_b5", "request", 512, 8, 4, 8, 8, mem=777, batch=5, m=15, n=18, faces=20, capacity=500, temperature=0.5, correct=64),
        # eight new sequences on the medium model: the one contraction that the matrix cores bound
        _case("admit_medium_b8", "admit", 1024, 16, 8, 16, 16, batch=8, capacity=2000),
        # new sequences whose memory is no whole number of tiles, heads of 96
        _case("admit_d768_ragged", "admit", 768, 8, 4, 8, 12, mem=1369, batch=2, m=15, n=18, capacity=1000),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    most = max(work(c)["bytes"] for c in listed() if c["kind"] == "step")
    while True:
        kind = rng.choice(["step", "step", "step", "request", "request", "admit"])
        c = _case("", kind, 0, 0, logint(2, 8), logint(2, 16), logint(2, 24))
        del c["name"]
        if rng.random() < 0.12:      # fp32: the small configurations only
            c.update(dtype="f32", bins=rng.choice([32, 128]), mem=logint(24, 600), batch=logint(1, 3))
            c["d"], c["heads"] = rng.choice([(128, 2), (192, 2), (256, 4), (256, 2)])
            c["c"], c["v"], c["f"] = min(c["c"], 4), min(c["v"], 4), min(c["f"], 6)
        else:
            c.update(bins=rng.choice([128, 1024, 1024]), mem=logint(100, 4096), batch=logint(1, 12))
            c["d"], c["heads"] = rng.choice([(256, 4), (512, 8), (512, 8), (768, 8), (768, 12), (1024, 8), (1024, 16), (1024, 16), (1536, 16), (1536, 24)])
            if rng.random() < 0.5:
                c["mem"] = max(256, c["mem"] // 256 * 256)
        c["c"], c["v"] = max(c["c"], 2), max(c["v"], 2)
        c["dc"], c["m"], c["n"] = rng.choice([(2, 9, 9), (2, 9, 9), (2, 15, 18), (2, 12, 18), (2, 9, 27), (3, 0, 0), (17, 0, 0)])
        if kind == "step":
            c["window"] = 9 * logint(20, 700)
        else:
            c["capacity"] = logint(50, 2000)
        if kind == "request":
            c["faces"] = logint(4, 24)
            c["speculative"] = rng.random() < 0.85
            c["temperature"] = rng.choice([0.0, 0.0, 0.5])
            c["correct"] = rng.choice([0, 0, 48]) if c["n"] else 0
        per = work(dict(c, kind="step", window=c["window"] or 9 * c["capacity"]))["bytes"]
        if per <= most and per * max(c["window"] / 9, 200) <= most * 500:
            return c


# -------------------------------------------------------------------------------------------- the model

def _block(c):
    return max(1 + c["dc"], c["m"], c["n"])


def _heads(c):
    """SP heads at the coordinate, vertex and face level; HF sets at the coordinate and vertex level."""
    return (c["dc"], max(c["m"] // 3 - 1, 0), max(c["n"] // 9 - 1, 0)), (max(max(c["m"], c["n"]) - 3, 0), max(c["n"] // 3 - 1, 0))


def _tensors(c):
    """(rows, columns) of every parameter tensor in the order of the blob; columns 0 = a gain vector."""
    d, V = c["d"], c["bins"] + 3
    sp, hf = _heads(c)
    block = [(d, 0)] + [(d, d)] * 4 + [(d, 0)] + [(d, d)] * 4 + [(d, 0), (4 * d, d), (d, 4 * d)]
    return ([(V, d)] + block * (c["c"] + c["v"] + c["f"]) + [(d, d)] * 2 + [(d, 0), (V, d)]
            + ([(d, 0)] + [(d, d)] * 5) * sum(sp) + [(d, 0), (d, d), (4 * d, d), (d, 4 * d)] * sum(hf) + [(3, d)])


def _cycle(bins):
    return np.random.default_rng(bins).permutation(bins)


@functools.lru_cache(maxsize=1)
def _blob(d, heads, c, v, f, bins, dtype, dc, m, n):
    """All parameters as one host array: the weights that a user's program has read from its checkpoint."""
    case = {"d": d, "c": c, "v": v, "f": f, "bins": bins, "dc": dc, "m": m, "n": n}
    shapes = _tensors(case)
    total = sum(r * max(k, 1) for r, k in shapes)
    gen = torch.Generator(device="cuda").manual_seed(20251115)
    w = torch.empty(total, device="cuda")
    for part in w.split(1 << 28):
        part.normal_(generator=gen)
    at, lm = 0, -1 - 6 * sum(_heads(case)[0]) - 4 * sum(_heads(case)[1]) - 1
    for i, (r, k) in enumerate(shapes):
        x = w[at:at + r * max(k, 1)]
        if i == 0:
            emb = x.mul_(4.0).view(r, k)
        elif k == 0:
            x.fill_(1.0)
        else:
            x.mul_(k ** -0.5)
            if i == len(shapes) + lm:
                cyc = torch.from_numpy(_cycle(bins)).cuda()
                x.view(r, k)[cyc.roll(-1)] = emb[cyc] * (0.25 * k ** -0.5)
        at += r * max(k, 1)
    if dtype == "bf16":
        for part in w.split(1 << 28):
            part.copy_(part.bfloat16())
    return w.cpu().numpy()


def _context(case):
    window = case["window"]
    cfg = FmConfig(d_model=case["d"], n_heads=case["heads"], ffn_mult=4, n_bins=case["bins"],
                   l_cpre=case["c"] // 2, l_cpost=case["c"] - case["c"] // 2, l_vpre=case["v"] // 2, l_vpost=case["v"] - case["v"] // 2,
                   l_face=case["f"], mem_len=case["mem"], dtype=1 if case["dtype"] == "bf16" else 0, max_batch=case["batch"],
                   max_tokens=9 * (STREAM_FACES if window else case["capacity"]), draft_coord=case["dc"], draft_point=case["m"],
                   draft_face=case["n"], hf_ffn_mult=4, ban_specials=1, rope_base=10000.0, rms_eps=1e-6, window=window, rules_off=0)
    fm = FlashMesh(cfg)
    fm.load_weights(_blob(*(case[k] for k in ("d", "heads", "c", "v", "f", "bins", "dtype", "dc", "m", "n"))))
    fm.set_sampling(case["temperature"], 11)
    fm.set_correct(case["correct"])
    return fm


# -------------------------------------------------------------------------------------------- a pass

def prepare(case, seed):
    """A context with its weights, the condition memories of the sequences, and the tokens each of them begins with."""
    fm = _context(case)
    S, B, bins = case["batch"], _block(case), case["bins"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    mems = list(torch.randn(S, case["mem"], case["d"], generator=gen, device="cuda"))
    # the stream of each sequence: the model's cycle from a random place (x_1 first), as long as the context holds
    start = torch.randint(0, bins, (S, 1), generator=gen, device="cuda")
    walk = torch.arange(fm.max_tokens, device="cuda")[None]
    cyc = torch.from_numpy(_cycle(bins)).cuda()
    stream = cyc[(start + walk) % bins].int().contiguous()
    first, first_len = fm.new_block()
    first[:, 0] = bins                                   # BOS
    first[:, 1:] = stream[:, :B - 1]
    first_len[:] = B
    tok, ln = fm.new_block()
    acc = torch.zeros(S, dtype=torch.int32, device="cuda")
    st = {"case": case, "fm": fm, "mems": mems, "first": first, "first_len": first_len, "tok": tok, "len": ln, "acc": acc,
          "logits": torch.zeros(S, B, bins + 3, device="cuda")}
    fm.set_draft_replay(stream, fm.max_tokens, 1.0, 0)
    if case["kind"] == "step":
        _begin(st)
        while int(fm.read_state()[:, 0].min()) < case["window"]:
            for _ in range(case["window"] // B + 2):     # fill the window: every draft right, one round as a rule
                _step(st)
    fm.set_draft_replay(stream, fm.max_tokens, KEEP, seed)
    return st


def _begin(st, logits=None):
    fm = st["fm"]
    for s, mem in enumerate(st["mems"]):
        fm.prefill_condition(s, mem)
    fm.verify_block(st["first"], st["first_len"], logits, st["acc"])
    fm.commit(st["first_len"])                           # the caller's own tokens: all of them are committed


def _step(st):
    fm = st["fm"]
    fm.draft(st["tok"], st["len"])
    fm.verify_block(st["tok"], st["len"], st["logits"], st["acc"])
    fm.commit(st["acc"])


def run(state):
    case, fm = state["case"], state["fm"]
    if case["kind"] == "step":
        _step(state)
        return {"logits": state["logits"], "block": state["tok"], "len": state["len"], "accepted": state["acc"]}
    if case["kind"] == "admit":
        _begin(state, state["logits"])
        return {"logits": state["logits"], "accepted": state["acc"]}
    _begin(state)
    tokens, count, _ = fm.generate(case["faces"], case["speculative"])
    return {"tokens": tokens, "count": count}


# -------------------------------------------------------------------------------------------- what a pass cannot do without

def work(case):
    c = case
    d, S, M, B = c["d"], c["batch"], c["mem"], _block(c)
    size = 2 if c["dtype"] == "bf16" else 4
    layers = (c["c"], c["v"], c["f"])
    nl, V = sum(layers), c["bins"] + 3
    sp, hf = _heads(c)
    backbone = nl * 14.0 * d * d + 2.0 * d * d + V * d
    heads = (5.0 * sum(sp) + 9.0 * sum(hf)) * d * d

    def step(context, block, draft):
        keys = (context, context / 3, context / 9)
        rows = (block, -(-block // 3), -(-block // 9))
        by = size * (backbone + (heads if draft else 0)) + size * 2.0 * d * S * sum(n * (k + M) for n, k in zip(layers, keys))
        fl = 2.0 * S * (sum(n * r * 14.0 * d * d for n, r in zip(layers, rows)) + rows[0] * V * d
                        + sum(n * r * 2.0 * d * (k + M) for n, r, k in zip(layers, rows, keys)) + (heads if draft else 0))
        return by + 4.0 * S * block * V, fl

    prefill = size * 2.0 * nl * d * d + S * (4.0 * M * d + size * nl * 2.0 * M * d), 4.0 * S * M * d * d * nl
    if c["kind"] == "step":
        by, fl = step(c["window"], B, True)
    else:
        by, fl = step(0, B, False)
        by, fl = by + prefill[0], fl + prefill[1]
    if c["kind"] == "request":
        tokens = 9 * c["faces"] - B
        steps = tokens if not c["speculative"] else tokens * (1 - KEEP) / (1 - KEEP ** B)
        one = step(4.5 * c["faces"], B if c["speculative"] else 1, c["speculative"])
        by, fl = by + steps * one[0], fl + steps * one[1]
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "request":
        return "exact"                                   # tokens, decided by clear margins
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 5e-3}
