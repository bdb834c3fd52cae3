"""Performance cases of the speculative-decoding engine: what a program that serves with it calls, over the sizes it
meets.

Kinds of case

  accept   the stand-alone accept / resample phase on the caller's logits (k_accept_static)
  request  one whole short request: prompt ingestion, then generation with a GammaTune controller per sequence
  step     one speculative step of a running generation: draft, verify, accept; the state moves on from pass to pass
  verify   one verification pass alone on a filled KV cache (the verification-only sweep)
  prefill  prompt ingestion through both models, then the first step, whose logits come back

Model pairs are those of synth.configs, by name and at full depth and width, with seeded random-init weights.  Greedy
pairs are used where logits come back, so that one rounding difference in a sampled draw does not change every later
value; drawing at a temperature is covered by `accept` (its inputs are given) and by `request` (a 32-bit pair).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2504_00030_amd as pk
import synth

ROOM = 1024  # tokens a running generation may grow by before it starts over from its prompt


def listed():
    return [
        # one accept phase in a serving loop: Vicuna-sized vocabulary, the usual four drafted tokens
        {"name": "accept-32k-k4", "kind": "accept", "vocab": 32000, "k": 4},
        # the same for a Llama-3-sized vocabulary at the largest speculation length of the 8B-shaped pair
        {"name": "accept-128k-k16", "kind": "accept", "vocab": 128256, "k": 16},
        # the smallest models: launches and host work only (prompt 32, 64 new tokens, temperature 1)
        {"name": "tiny-request", "kind": "request", "pair": "tiny", "batch": 1, "prompt": 32, "generate": 64},
        # single-stream decoding with a small target and a two-layer draft, plain acceptance
        {"name": "1b-step", "kind": "step", "pair": "1b", "batch": 1, "context": 256, "gamma": 4, "uneven": False, "stop": False},
        # single-stream decoding of the 7B-shaped pair
        {"name": "7b-step", "kind": "step", "pair": "7b", "batch": 1, "context": 512, "gamma": 5, "uneven": False, "stop": False},
        # the headline: 8B-shaped pair, one sequence, its mean speculation length of 2, early stopping armed
        {"name": "8b-step", "kind": "step", "pair": "8b", "batch": 1, "context": 1024, "gamma": 2, "uneven": False, "stop": True},
        # four sequences decoding in lock-step, each with a speculation length of its own
        {"name": "8b-batch4-step", "kind": "step", "pair": "8b", "batch": 4, "context": 1024, "gamma": 4, "uneven": True, "stop": False},
        # 8-bit weights, a longer speculation
        {"name": "8b-q8-step", "kind": "step", "pair": "8b-q8", "batch": 1, "context": 777, "gamma": 6, "uneven": False, "stop": False},
        # many sequences in lock-step: the verification pass of 32 sequences that drafted two tokens each
        {"name": "7b-batch32-verify", "kind": "verify", "pair": "7b", "batch": 32, "kv": 512, "rows": 3},
        # a cell of the 13B-shaped verification sweep: four sequences, eight rows each
        {"name": "13b-verify", "kind": "verify", "pair": "13b", "batch": 4, "kv": 2048, "rows": 8},
        # the headline's prompt: 1024 tokens into both models
        {"name": "8b-prefill", "kind": "prefill", "pair": "8b", "batch": 1, "prompt": 1024},
        # short prompts of different lengths arriving together
        {"name": "7b-prefill-ragged", "kind": "prefill", "pair": "7b", "batch": 4, "prompt": 117},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["accept", "request", "step", "step", "step", "verify", "verify", "prefill", "prefill"])
    if kind == "accept":
        return {"kind": kind, "vocab": _log_int(rng, 4000, 128256), "k": rng.randint(1, 16)}
    if kind == "request":
        return {"kind": kind, "pair": "tiny", "batch": rng.randint(1, 3), "prompt": rng.randint(5, 64), "generate": rng.randint(24, 96)}
    if kind == "step":
        pair = rng.choice(["1b", "7b", "8b", "8b", "8b-q8"])
        batch = rng.choice([1, 1, 2, 3, 4, 6])
        return {"kind": kind, "pair": pair, "batch": batch, "context": _log_int(rng, 40, 1200), "gamma": rng.randint(1, 12 // min(batch, 3)),
                "uneven": batch > 1 and rng.random() < 0.5, "stop": rng.random() < 0.5}
    if kind == "verify":
        pair = rng.choice(["7b", "8b", "8b-q8", "13b"])
        batch = _log_int(rng, 1, 8 if pair == "13b" else 32)
        return {"kind": kind, "pair": pair, "batch": batch, "kv": _log_int(rng, 100, 2048 if batch <= 8 else 1024),
                "rows": rng.randint(1, max(1, min(16, 100 // batch)))}
    pair = rng.choice(["1b", "7b", "8b", "8b-q8"])
    batch = rng.randint(1, 6)
    return {"kind": "prefill", "pair": pair, "batch": batch, "prompt": max(3, _log_int(rng, 40, 1024) // batch)}


def _ragged_lengths(n, batch):
    """Prompt lengths of one arrival: the longest is n, the others fall off unevenly."""
    return [max(1, n - (b * n) // (2 * batch) - (b % 3)) for b in range(batch)]


def _gammas(case):
    """Planned speculation lengths of a step, one per sequence."""
    b, g = case["batch"], case["gamma"]
    return np.array([max(1, g - (i % 4)) if case["uneven"] else g for i in range(b)], dtype=np.int32)


def _engine(cfg, case, seed, **kw):
    Wt, Wd = synth.make_pair_weights(cfg, seed, device="cuda")
    torch.cuda.synchronize()
    return pk.SpecEngine(cfg.target, Wt, cfg.draft, Wd, batch=case["batch"], seed=seed, use_graphs=True, **kw)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "accept":
        # target and draft logits that agree as a draft model's do: N(0, 2) draft logits, the target's a noisy copy
        gen = torch.Generator(device="cuda").manual_seed(seed)
        k, v = case["k"], case["vocab"]
        q = 2.0 * torch.randn((k, v), generator=gen, device="cuda")
        p = 2.0 * torch.randn((k + 1, v), generator=gen, device="cuda")
        p[:k] = 0.8 * q + 0.6 * p[:k]
        drafted = torch.multinomial(torch.softmax(q, dim=1), 1, generator=gen).reshape(k).to(torch.int32)
        return {"case": case, "seed": seed, "p": p, "q": q, "drafted": drafted,
                "result": torch.zeros(2, dtype=torch.int32, device="cuda")}
    cfg = synth.pair(case["pair"])
    if kind == "request":
        prompts = synth.make_prompts(case["batch"], case["prompt"], cfg.target.vocab, seed)
        eng = _engine(cfg, case, seed, max_seq=case["prompt"] + 3 * case["generate"] + cfg.gamma_max + 2, gamma_max=cfg.gamma_max,
                      temperature=1.0)
        return {"case": case, "eng": eng, "prompts": prompts, "gamma_max": cfg.gamma_max}
    if kind == "step":
        # the 1B-shaped pair accepts by the real test; the others are driven by the forced landscape: everything
        # accepted where early stopping is armed (no draft pass is cut short), else six tokens in ten
        natural = case["pair"] == "1b"
        eng = _engine(cfg, case, seed, max_seq=case["context"] + ROOM, gamma_max=max(cfg.gamma_max, case["gamma"]), temperature=0.0,
                      accept_mode=pk.ACCEPT_NATURAL if natural else pk.ACCEPT_FORCED)
        if not natural:
            eng.set_forced_alpha(synth.alpha_constant(1.0 if case["stop"] else 0.6, 1))
        if case["stop"]:
            eng.set_early_stop(0.0001 if natural else 0.4)
        prompts = synth.make_prompts(case["batch"], case["context"], cfg.target.vocab, seed)
        eng.prefill(prompts)
        return {"case": case, "eng": eng, "prompts": prompts, "len": np.full(case["batch"], case["context"], dtype=np.int64)}
    if kind == "verify":
        cfg = synth.shrink(cfg, cfg.target.n_layers, 1)  # the draft model has no part in it
        eng = _engine(cfg, case, seed, max_seq=case["kv"] + 40, gamma_max=max(1, case["rows"] - 1), temperature=1.0)
        eng.fill_kv(case["kv"], seed)
        return {"case": case, "eng": eng}
    n = case["prompt"]
    lens = _ragged_lengths(n, case["batch"])
    prompts = [synth.make_prompts(1, m, cfg.target.vocab, seed + 1000 * b)[0].tolist() for b, m in enumerate(lens)]
    eng = _engine(cfg, case, seed, max_seq=n + 64, gamma_max=cfg.gamma_max, temperature=0.0)
    return {"case": case, "eng": eng, "prompts": prompts}


def _texts(eng, room):
    """The text so far of every sequence, in rows of one length."""
    rows = np.zeros((eng.batch, room), dtype=np.int32)
    for b in range(eng.batch):
        t = eng.read_tokens(b)
        rows[b, : len(t)] = t
    return rows


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "accept":
        pk.k_accept_static(state["p"], state["q"], state["drafted"], 1.0, state["seed"], 3, state["result"])
        return state["result"]
    eng = state["eng"]
    if kind == "request":
        eng.prefill(state["prompts"])
        ctrls = [pk.GammaTune(eta=0.25, delta=1, gamma_min=1, gamma_max=state["gamma_max"], gamma0=4) for _ in range(case["batch"])]
        st = eng.run(case["generate"], ctrls)
        return {"tokens": [eng.read_tokens(b)[: case["prompt"] + case["generate"]] for b in range(case["batch"])],
                "steps": st["spec_steps"], "accepted": st["accepted"], "drafted": st["drafted"],
                "gamma": [c.gamma for c in ctrls], "gamma_bar": [c.gamma_bar for c in ctrls]}
    if kind == "step":
        g = case["gamma"]
        if int(state["len"].max()) + g + 1 > case["context"] + ROOM:  # full: the next request starts
            eng.prefill(state["prompts"])
            state["len"][:] = case["context"]
        gs = _gammas(case)
        eng.draft(gs if case["batch"] > 1 else g)
        eng.verify(int(gs.max()))
        A, y, k = eng.accept()
        state["len"] += A + 1
        return {"accepted": A, "drafted": k, "tokens": _texts(eng, case["context"] + ROOM),
                "logits": eng.debug_logits(1)}
    if kind == "verify":
        eng.verify_rows(case["rows"])
        return {"logits": eng.debug_logits(1)}
    eng.prefill_ragged(state["prompts"])
    eng.draft(1)
    eng.verify(1)
    A, y, k = eng.accept()
    return {"accepted": A, "drafted": k, "tokens": _texts(eng, case["prompt"] + 64),
            "draft_logits": eng.debug_logits(0), "logits": eng.debug_logits(1)}


def _weights(m):
    """(bytes, parameters) of the layers and of the LM head of one model."""
    one = {"bf16": 2, "q8": 1}.get(m.dtype, 4)
    head = m.vocab * m.d_model
    body = m.n_params() - head
    return body * one, body, head * one, head


def _pass_work(m, rows, contexts, out_rows):
    """Bytes and operations of one forward pass: every weight once, the cached keys and values of `contexts` positions,
    the logits of `out_rows` rows written."""
    bb, bp, hb, hp = _weights(m)
    att = 4.0 * m.n_layers * m.n_q_heads * m.head_dim * sum(contexts) * (rows / max(1, len(contexts)))
    b = bb + m.kv_bytes_per_token() * sum(contexts)
    f = 2.0 * bp * rows + att
    if out_rows:
        b += hb + 4.0 * out_rows * m.vocab
        f += 2.0 * hp * out_rows
    return b, f


def work(case):
    kind = case["kind"]
    if kind == "accept":
        k, v = case["k"], case["vocab"]
        return {"bytes": 4.0 * v * (2 * k + 1) + 4 * k + 8, "flops": 5.0 * v * (2 * k + 1)}
    cfg = synth.pair(case["pair"])
    t, d = cfg.target, cfg.draft
    B = case["batch"]
    total_b = total_f = 0.0

    def add(w, times=1):
        nonlocal total_b, total_f
        total_b += times * w[0]
        total_f += times * w[1]

    if kind == "request":
        n, g = case["prompt"], cfg.gamma_max
        steps = math.ceil(case["generate"] / (g + 1))  # the least number of steps: everything accepted
        for m in (t, d):
            add(_pass_work(m, B * n, [n // 2] * B, 0))
        add(_pass_work(d, B, [n] * B, B), steps * g)
        add(_pass_work(t, B * (g + 1), [n] * B, B * (g + 1)), steps)
    elif kind == "step":
        gs = _gammas(case)
        for j in range(int(gs.max())):
            live = int((gs > j).sum())
            add(_pass_work(d, live, [case["context"]] * live, live))
        rows = int((gs + 1).sum())
        add(_pass_work(t, rows, [case["context"]] * B, rows))
    elif kind == "verify":
        rows = B * case["rows"]
        add(_pass_work(t, rows, [case["kv"]] * B, rows))
    else:
        lens = _ragged_lengths(case["prompt"], B)
        rows = sum(lens)
        for m in (t, d):
            bb, bp, _, _ = _weights(m)
            att = sum(2.0 * m.n_layers * m.n_q_heads * m.head_dim * n * n for n in lens)  # causal: half the square
            add((bb + m.kv_bytes_per_token() * rows, 2.0 * bp * rows + att))
        add(_pass_work(d, B, lens, B))
        add(_pass_work(t, 2 * B, lens, 2 * B))
    return {"bytes": total_b, "flops": total_f}


def tolerance(case):
    # accept returns whole numbers, from sums in 64 bits
    if case["kind"] == "accept":
        return "exact"
    # a 32-bit pair: tokens, counts and the controllers' averages of whole numbers
    if case["kind"] == "request":
        return {"rel": 1e-5}
    # Logits of deep 16-bit models.  The same weights with the attention cut into chunks of another size and the down
    # projections summed in another order: rel 1.6e-4 (1B), 3.5e-4 to 4.4e-4 (8B, 16- and 8-bit), 5.4e-4 (7B), 1.6e-3
    # (7B after its prompt's ingestion); max 7e-4 to 7.3e-3.  A token may turn at a near tie of two logits.
    return {"rel": 6e-3, "max": 0.03, "differ": 0.01}
