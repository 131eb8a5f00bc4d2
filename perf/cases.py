"""The work that users of this framework have it do, as measurable cases.

Every case is one pass through the public entry points of paper_2405_01481_amd.rollout over one of the model
shapes of paper_2405_01481_amd.synth.  Shapes keep their full width; where the depth would make a pass take seconds
it is cut (every layer does the same work), as the repository's own tests do for the 70B shape.

kinds
  step      one PPO rollout step: rollout_refresh_policy (the weights have just been updated in place),
            rollout_generate, score_logprobs_kl of prompt + response under policy and reference, ppo_rewards
  generate  rollout_generate alone: prefill of the prompts and `gen` decode steps
  queue     rollout_generate_queue: more prompts than slots, per-prompt limits, end-of-sequence tokens
  score     score_logprobs_kl alone (the log-probs stage: policy and reference)
  kl_exact  score_kl_exact: the full-vocabulary KL of both models
  values    score_values of a critic / reward model, then ppo_rewards with the sequence scores

Sequence lengths are ragged between `lo` and `hi` where a case has both.  `copies`: the caller gives the policy
(and the reference) a buffer for the library's fp16 copy, as bench.py does when there is room.
"""
import contextlib
import math

import numpy as np
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

DEV = "cuda:0"
SHAPES = {"tiny": synth.TINY, "1b": synth.L1B, "8b": synth.L8B, "70b": synth.L70B}
KL_COEF = 0.003                  # Section 3.3


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest user: the fp32 configuration's whole step, one token at a time -- launches and latency count
        dict(name="step_tiny_fp32", kind="step", shape="tiny", layers=2, batch=4, lo=32, hi=32, gen=32, temp=0.0, copies=False),
        # the 1B configuration's step, shorter response
        dict(name="step_1b", kind="step", shape="1b", layers=16, batch=64, lo=256, hi=256, gen=48, temp=0.3, copies=True),
        # a handful of ragged prompts at full 8B depth: what somebody who looks at single answers waits for
        dict(name="generate_8b_few", kind="generate", shape="8b", layers=32, batch=3, lo=25, hi=190, gen=24, temp=0.3, copies=True),
        # the headline's batch and prompt length: 128 rows, all decode kernels at their widest
        dict(name="generate_8b", kind="generate", shape="8b", layers=8, batch=128, lo=512, hi=512, gen=160, temp=0.0, copies=True),
        # long ragged prompts, long contexts in decode
        dict(name="generate_8b_long", kind="generate", shape="8b", layers=8, batch=32, lo=1024, hi=2048, gen=96, temp=0.0, copies=True),
        # 70B width: the weights fill the device, so there is no fp16 copy
        dict(name="generate_70b", kind="generate", shape="70b", layers=4, batch=64, lo=100, hi=300, gen=48, temp=0.0, copies=False),
        # dynamic slots: refills prefill a few short prompts at a time between decode bursts
        dict(name="queue_1b", kind="queue", shape="1b", layers=16, batch=32, prompts=80, lo=40, hi=256, gen=96, temp=0.0, copies=True),
        # the log-probs stage at the headline's sequence length
        dict(name="score_8b", kind="score", shape="8b", layers=8, batch=32, lo=1024, hi=1024, copies=True),
        # the paper's micro-batch of 8 on a smaller model, ragged
        dict(name="score_1b_micro", kind="score", shape="1b", layers=16, batch=8, lo=70, hi=512, copies=True),
        # 70B width, long ragged sequences, weights converted in the kernels
        dict(name="score_70b_long", kind="score", shape="70b", layers=4, batch=5, lo=1500, hi=4096, copies=False),
        # exact KL of both models over the whole vocabulary
        dict(name="kl_exact_8b", kind="kl_exact", shape="8b", layers=4, batch=8, lo=300, hi=1024, copies=True),
        # critic values and rewards of one micro-batch
        dict(name="values_8b", kind="values", shape="8b", layers=8, batch=8, lo=200, hi=1000, copies=False),
    ]


# What a drawn case may be: kind, shape, range of layers, batch, sequence length, generated tokens.
_RANGES = [
    ("step", "tiny", (2, 2), (1, 8), (8, 64), (8, 48)),
    ("step", "1b", (16, 16), (4, 64), (16, 256), (8, 64)),
    ("generate", "8b", (32, 32), (1, 8), (16, 256), (8, 24)),
    ("generate", "8b", (8, 8), (8, 128), (64, 2048), (8, 160)),
    ("generate", "70b", (4, 4), (4, 64), (32, 1024), (8, 48)),
    ("queue", "1b", (16, 16), (8, 48), (16, 256), (16, 96)),
    ("score", "1b", (16, 16), (1, 64), (64, 512), None),
    ("score", "8b", (8, 8), (1, 32), (128, 4096), None),
    ("score", "70b", (4, 4), (1, 8), (256, 4096), None),
    ("kl_exact", "8b", (4, 4), (1, 8), (64, 1024), None),
    ("values", "8b", (8, 8), (1, 32), (64, 1024), None),
]


def _log_int(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(case):
    """Rough seconds of a pass: only to keep drawn cases below the largest listed one."""
    w = work(case)
    steps = case.get("gen", 0) * (3 if case["kind"] == "queue" else 1)
    return w["bytes"] / 3e12 + w["flops"] / 8e14 + steps * case["layers"] * 5e-5


def draw(rng):
    cap = 0.8 * max(_cost(c) for c in listed())
    while True:
        kind, shape, layers, batch, length, gen = rng.choice(_RANGES)
        c = dict(kind=kind, shape=shape, layers=rng.randint(*layers), batch=_log_int(rng, *batch))
        c["hi"] = _log_int(rng, *length)
        c["lo"] = c["hi"] if kind != "step" and rng.random() < 0.2 else max(1, int(c["hi"] * rng.uniform(0.2, 1.0)))
        if kind == "step":
            c["lo"] = c["hi"]
        if gen:
            c["gen"] = _log_int(rng, *gen)
            # a uniform number within rounding of a step of the distribution function picks either token, and the row
            # goes its own way from there: about one draw in 1e5, so long large batches are greedy
            c["temp"] = 0.0 if shape == "tiny" or kind == "queue" or c["batch"] * c["gen"] > 2500 or rng.random() < 0.3 else 0.3
        if kind == "queue":
            c["prompts"] = int(c["batch"] * rng.uniform(1.2, 3.0)) + 1
        c["copies"] = shape in ("1b", "8b") and kind != "values" and rng.random() < 0.75
        if _cost(c) <= cap:
            return c


# ------------------------------------------------------------------------------------------------ inputs
def _shape(case):
    base = SHAPES[case["shape"]]
    return base if case["layers"] == base.n_layers else synth.scaled_shape(base, base.name, n_layers=case["layers"])


def _lengths(case, n):
    """Ragged lengths, the same for every seed: a deterministic spread over [lo, hi] with both ends in it."""
    lo, hi = case["lo"], case["hi"]
    if lo == hi or n == 1:
        return np.full(n, hi, np.int32)
    r = np.random.default_rng(1000 * n + lo + hi)
    x = r.integers(lo, hi + 1, size=n)
    x[0], x[-1] = hi, lo
    return x.astype(np.int32)


def _predictive(w, s):
    """Give a random-weight policy next-token distributions of a trained model's kind -- one continuation clearly
    ahead of the rest (most of the probability) -- instead of a near-uniform one over the whole vocabulary, whose
    draws hang on the last bit of every sum: token v is followed by v + 1.  The embedding is scaled up until it is
    about as large as what the layers add to it, and the LM head's row v + 1 leans towards it."""
    d = s.d_model
    g = s.w_std * math.sqrt(d)                                      # std of gate and up
    act = g * 0.5 * g * math.sqrt(1.0 + 0.75 * g * g)               # rms of silu(gate) * up
    out = s.w_std * math.sqrt(s.d_ffn) * act * math.sqrt(s.n_layers)   # what the layers add to the residual stream
    a = max(out, s.w_std)
    lead = 0.85 * math.log(s.vocab) + 6.0                           # logit of the continuation
    cos = a / math.hypot(a, out)
    emb, head = w["tok_embed"], w["lm_head"]
    step = max(1, (1 << 27) // d)
    for r0 in range(0, s.vocab, step):
        emb[r0:r0 + step] = (emb[r0:r0 + step].float() * (a / s.w_std)).to(emb.dtype)
    b = lead / (a * d * cos)
    for r0 in range(0, s.vocab, step):
        idx = torch.arange(r0 - 1, min(r0 + step, s.vocab) - 1, device=emb.device) % s.vocab
        head[r0:r0 + step] = (head[r0:r0 + step].float() + emb[idx].float() * b).to(head.dtype)


def _weights(s, seed, cfg, copies, predictive):
    w = synth.make_weights(s, seed, DEV)
    if predictive:
        _predictive(w, s)
    shadow = torch.empty(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV) if copies else None
    return R.Weights(w, shadow=shadow)


def _tokens(rows, width, vocab, lens, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    ids = torch.randint(0, vocab, (rows, width), generator=g, dtype=torch.int32, device=DEV)
    ids[torch.arange(width, device=DEV)[None, :] >= torch.tensor(lens, device=DEV)[:, None]] = 0
    return ids


_stream = None


def _side_stream():
    """Generation replays a captured step, which needs a stream of its own; a program keeps one."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def prepare(case, seed):
    seed = int(seed)
    s, kind, B = _shape(case), case["kind"], case["batch"]
    gen = case.get("gen", 0)
    Lmax = case["hi"] + gen
    cfg = R.make_cfg(s, B, max(Lmax, 2))
    pw = _weights(s, 4 * seed + 1, cfg, case["copies"], kind in ("step", "generate", "queue"))
    st = dict(case=case, shape=s, policy=pw, stream=_side_stream())
    if kind in ("step", "score", "kl_exact"):
        st["reference"] = _weights(s, 4 * seed + 2, cfg, case["copies"], False)
    st["ro"] = R.Rollout(cfg, pw, DEV)
    z = lambda *sh, dt=torch.float32: torch.zeros(*sh, dtype=dt, device=DEV)   # noqa: E731
    if kind in ("step", "generate", "queue"):
        n = case.get("prompts", B)
        lens = _lengths(case, n)
        st["ids"], st["plen"] = _tokens(n, case["hi"], s.vocab, lens, 4 * seed + 3), lens
        st["out"], st["olen"], st["olp"] = z(n, gen, dt=torch.int32), z(n, dt=torch.int32), z(n, gen)
        st["sample"] = R.sample_cfg(seed, case["temp"])
    if kind == "queue":
        # log-normal response lengths, as the benchmark's queue workload; half of the rows end by the
        # end-of-sequence token (the continuation of token v is v + 1), the others by their limit
        r = np.random.default_rng(7 * n + gen)
        want = np.clip(np.rint(r.lognormal(math.log(0.45 * gen), 0.7, n)), min(4, gen), gen).astype(np.int32)
        eos = s.vocab - 5
        st["limit"] = want.copy()
        for q in range(0, n, 2):
            st["limit"][q] = gen
            st["ids"][q, int(lens[q]) - 1] = eos - int(want[q])
        st["sample"] = R.sample_cfg(seed, case["temp"], eos)
    if kind in ("step", "score", "kl_exact", "values"):
        if kind == "step":
            st["full"] = z(B, Lmax, dt=torch.int32)
            st["slen"] = (st["plen"] + gen).astype(np.int32)
        else:
            st["slen"] = _lengths(case, B)
            st["plen"] = np.maximum(1, st["slen"] // 2).astype(np.int32)
            st["full"] = _tokens(B, case["hi"], s.vocab, st["slen"], 4 * seed + 3)
        st["scores"] = [z(B, Lmax) for _ in range(4)]
        st["rewards"] = z(B, Lmax)
    if kind in ("step", "values"):
        g = torch.Generator(device=DEV)
        g.manual_seed(4 * seed + 4)
        st["head"] = (torch.randn(s.d_model, generator=g, device=DEV) * 0.05).to(s.torch_dtype)
        st["seq_reward"] = torch.randn(B, generator=g, device=DEV)
        st["kl"] = torch.randn(B, Lmax, generator=g, device=DEV)
        st["last"] = torch.tensor(st["slen"] - 1, dtype=torch.int64, device=DEV)[:, None]
    return st


# ------------------------------------------------------------------------------------------------ one pass
def run(st):
    case, ro, kind = st["case"], st["ro"], st["case"]["kind"]
    with torch.cuda.stream(st["stream"]):
        if kind == "generate":
            ro.rollout_generate(st["sample"], st["ids"], st["plen"], case["gen"], st["out"], st["olen"], st["olp"])
            return st["out"], st["olen"], st["olp"]
        if kind == "queue":
            ro.rollout_generate_queue(st["sample"], st["ids"], st["plen"], st["limit"], case["gen"], st["out"], st["olen"],
                                      st["olp"])
            return st["out"], st["olen"], st["olp"]
        if kind == "step":
            ro.rollout_refresh_policy()
            ro.rollout_generate(st["sample"], st["ids"], st["plen"], case["gen"], st["out"], st["olen"], st["olp"])
            P = case["hi"]
            st["full"][:, :P] = st["ids"]
            st["full"][:, P:] = st["out"]
            ro.score_logprobs_kl(st["policy"], st["reference"], st["full"], st["slen"], st["plen"], KL_COEF, *st["scores"])
            ro.ppo_rewards(st["scores"][2], st["seq_reward"], st["slen"], st["plen"], KL_COEF, st["rewards"])
            return [st["out"], st["olen"], st["olp"], st["rewards"]] + st["scores"]
        if kind == "score":
            ro.score_logprobs_kl(st["policy"], st["reference"], st["full"], st["slen"], st["plen"], KL_COEF, *st["scores"])
            return st["scores"]
        if kind == "kl_exact":
            ro.score_kl_exact(st["policy"], st["reference"], st["full"], st["slen"], st["plen"], st["scores"][0])
            return st["scores"][0]
        ro.score_values(st["policy"], st["head"], st["full"], st["slen"], st["scores"][0])
        ro.ppo_rewards(st["kl"], st["scores"][0].gather(1, st["last"])[:, 0].contiguous(), st["slen"], st["plen"], KL_COEF,
                       st["rewards"])
        return st["scores"][0], st["rewards"]


# ------------------------------------------------------------------------------------------------ work, tolerance
def work(case):
    """Bytes: the weights a pass reads (once per decode step, since a step needs the token before it and no cache
    holds a model; once per scored model otherwise), the KV cache read and written in decode, ids in and results out.
    Operations: two per weight and token (the LM head only where a token is drawn or scored), and the attention
    products of the causal triangle."""
    s, kind, B = _shape(case), case["kind"], case["batch"]
    e = 4 if s.dtype == "fp32" else 2
    body, head = s.body_params(), s.head_params()
    att = 4.0 * s.n_layers * s.n_q_heads * s.head_dim                # flops per (query, key) pair
    kvt = s.kv_bytes_per_token()
    gen = case.get("gen", 0)
    byts = flops = 0.0
    tri = lambda n: n * (n + 1) / 2.0                                # noqa: E731
    if kind in ("step", "generate", "queue"):
        n = case.get("prompts", B)
        lens = _lengths(case, n).astype(float)
        g = np.full(n, float(gen))
        if kind == "queue":
            r = np.random.default_rng(7 * n + gen)
            g = np.clip(np.rint(r.lognormal(math.log(0.45 * gen), 0.7, n)), min(4, gen), gen)
        steps = max(float(g.max()), float(g.sum()) / B)
        pre = lens - 1
        flops += 2.0 * body * pre.sum() + att * tri(pre).sum() + 2.0 * (body + head) * g.sum()
        flops += att * (g * lens + tri(g)).sum()
        byts += e * body + steps * e * (body + head)                  # prefill, then one sweep per step
        byts += kvt * (pre.sum() + (g * (lens + 1) + tri(g)).sum())   # cache written by prefill; read and extended per step
        byts += 4.0 * lens.sum() + 8.0 * g.sum() + 2.0 * e * s.d_model * g.sum()
    if kind in ("step", "score", "kl_exact", "values"):
        models = 1 if kind == "values" else 2
        L = (_lengths(case, B) + gen).astype(float)
        flops += models * (2.0 * body * L.sum() + att * tri(L).sum())
        if kind != "values":
            flops += models * 2.0 * head * (L - (L // 2 if kind == "kl_exact" else 1)).sum()
        byts += models * e * (body + (head if kind != "values" else 0))
        byts += models * e * s.d_model * L.sum() + 4.0 * L.sum() * (1 + 4)
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """Measured: fp32 sums in another order; bf16 shapes with another number of fp16-pair layers, with logits instead of
    block statistics in the sampler, and on the plain kernels.  Largest relative errors seen, over all outputs of a
    kind: log-probs and KL of scoring 2.1e-3 (max 1.3e-2), log-probs of generation 8.6e-4 (max 3e-3; they are small
    numbers, see _predictive), exact KL 2.9e-5 (max 1.1e-4), values and rewards 4.6e-3 (max 5.3e-2)."""
    if case["shape"] == "tiny":
        return {"rel": 2e-4, "max": 2e-3, "differ": 0.0}
    rel, most = {"values": (1.8e-2, 0.2), "kl_exact": (2e-4, 1e-3), "score": (8e-3, 5e-2)}.get(case["kind"], (4e-3, 1.5e-2))
    if case["kind"] == "step":
        rel, most = 8e-3, 5e-2
    return {"rel": rel, "max": most, "differ": 0.005}
