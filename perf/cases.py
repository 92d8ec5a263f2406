"""Workloads of the draft -> verify -> accept engine: what a decoding program asks of it, call by call.

Every case is one pass through `Engine`'s public calls on synthetic models of the repository's own widths
(`synth`).  Kinds:

* ``step``    one speculative decoding step: sf_draft_step, sf_verify_step, sf_accept_commit;
* ``plain``   one step of plain greedy decoding (k = 0: sf_verify_step, sf_accept_commit);
* ``prefill`` Engine.prefill of a ragged batch of prompts in blocks of ``block`` tokens;
* ``draft``   sf_draft_step alone in the two-stage wiring (context attention and slot attention apart).

The wide models are run at a part of their depth (their layers are alike), so that several states fit the card.

The models are random-init with one regularity planted, as trained models have and random ones lack: the
embedding dominates the residual stream and the LM head's row of token v + 1 looks along the embedding of
token v, so the greedy choice has a clear lead everywhere and does not hang on rounding.  Drafted tokens handed
to the verify pass are the target's own continuation with each slot corrupted often enough that about 1.75 tokens
are accepted per call, which is what the draft of a trained model of this class reaches.
"""
import math
import random

import torch

import synth
from paper_2511_20340_amd import binding as sfb
from paper_2511_20340_amd.engine import Engine

MODELS = {"tiny": synth.TINY, "1b": synth.M1B, "8b": synth.M8B, "14b": synth.M14B}
EMBED_STD = 16.0       # of the embedding rows; 40 layers add a residual of about 11
ACCEPT_PROB = 0.438    # per slot: 1 + a + a^2 + a^3 + a^4 = 1.75


def listed():
    def case(name, kind, model, layers, batch, lo, hi, k, **more):
        c = {"name": name, "kind": kind, "model": model, "layers": layers, "batch": batch, "lo": lo, "hi": hi, "k": k,
             "logits": True, "graph": False, "mask": "bidir"}
        c.update(more)
        return c
    return [
        # the fp32 mode of small models: the step is nothing but launches
        case("tiny_f32_step", "step", "tiny", 2, 4, 64, 64, 4),
        # one user at a terminal: a single sequence, latency counts
        case("1b_single_step", "step", "1b", 16, 1, 700, 700, 4),
        # the small model's batch, one graph replay per step as a serving loop has it; logits are not kept
        case("1b_step_graph", "step", "1b", 16, 32, 512, 512, 4, graph=True, logits=False),
        # mid-size model, ragged batch of 64
        case("8b_step_b64", "step", "8b", 16, 64, 256, 2048, 4),
        # throughput serving: 256 sequences of one length
        case("8b_step_b256", "step", "8b", 16, 256, 1024, 1024, 4, logits=False),
        # the largest single-GPU workload: 128 ragged sequences of 1024 to 4096 tokens
        case("14b_step_b128", "step", "14b", 20, 128, 1024, 4096, 4, graph=True, logits=False),
        # plain decoding of an odd-sized batch, the "without speculation" row of every comparison
        case("8b_plain_b61", "plain", "8b", 16, 61, 100, 1800, 0),
        # a few users with long documents: the key/value read is split over the chip
        case("8b_long_context", "step", "8b", 8, 3, 9000, 16000, 4),
        # longer drafts (k = 7, causal block mask) on an odd batch
        case("8b_step_k7", "step", "8b", 8, 17, 130, 1500, 7, mask="causal"),
        # prompt ingestion of a ragged batch in 64-token blocks
        case("1b_prefill", "prefill", "1b", 16, 8, 100, 900, 4, block=64),
        # the paper's two attentions kept apart, drafting alone
        case("14b_two_stage_draft", "draft", "14b", 1, 96, 512, 2048, 4),
    ]


def draw(rng):
    """One more case of the same ranges; its work stays below that of the largest listed one."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.choice(["step", "step", "step", "step", "plain", "prefill", "draft"])
    model = rng.choice(["1b", "8b", "14b", "1b", "8b", "14b", "tiny"]) if kind == "step" else rng.choice(["1b", "8b", "14b"])
    layers = {"tiny": 2, "1b": 16, "8b": 8, "14b": 6}[model]
    k = {"step": rng.randint(1, 8), "draft": rng.randint(1, 8), "plain": 0, "prefill": 4}[kind]
    if kind == "prefill":
        layers = {"1b": 16, "8b": 4, "14b": 3}[model]
        batch, hi = log_int(1, 12), log_int(65, 1000)
        lo = max(1, hi // rng.randint(1, 6))
    elif model == "tiny":
        batch, hi = log_int(1, 16), log_int(16, 400)
        lo = max(1, hi // rng.randint(1, 4))
    else:
        batch = log_int(1, {"1b": 128, "8b": 256, "14b": 128}[model])
        room = 4000000 // (batch * layers)        # bounds the caches at about 16 GB
        hi = min(log_int(64, 8192), max(64, room))
        lo = max(1, hi // rng.randint(1, 6))
    if kind == "draft":
        layers = 1
    c = {"kind": kind, "model": model, "layers": layers, "batch": batch, "lo": lo, "hi": hi, "k": k,
         "logits": kind != "prefill" and rng.random() < 0.5, "graph": kind == "step" and rng.random() < 0.3,
         "mask": rng.choice(["bidir", "bidir", "causal"])}
    if kind == "prefill":
        c["block"] = rng.choice([16, 32, 64, 128 if model == "1b" else 64])
    return c


def _shape(case):
    return MODELS[case["model"]].scaled(n_layers=case["layers"])


def _lengths(case, seed):
    r = random.Random(seed * 7919 + 17)
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]


def _weights(m, k, seed, two_stage):
    """synth.device_weights with the planted successor rule (see the top of the file)."""
    tw, dw = synth.device_weights(m, k, seed, two_stage)
    d = m.d_model
    tw["lm_head"] = torch.roll(tw["embed"], 1, 0)          # row v + 1 looks along the embedding of v
    tw["embed"] = tw["embed"] * (EMBED_STD / 0.02)
    eye = torch.arange(d, device="cuda")
    dw["w_ds"][eye, eye] += 4.0                            # the draft state keeps the embedding too ...
    for s in range(k):
        dw["w_pos"][s * d + eye, eye] += 4.0               # ... and so does every slot
    return tw, dw


def _uniform(shape, lo, hi, g, dtype=torch.int32):
    return torch.randint(lo, hi, shape, generator=g, device="cuda", dtype=dtype)


class _State:
    pass


def prepare(case, seed):
    m, B, k, kind = _shape(case), case["batch"], case["k"], case["kind"]
    s = _State()
    s.case, s.k = case, k
    s.mask = sfb.SF_MASK_BIDIR if case["mask"] == "bidir" else sfb.SF_MASK_CAUSAL
    if kind == "draft":
        s.mask |= sfb.SF_DRAFT_TWO_STAGE
    lens = _lengths(case, seed)
    cap = synth.kv_capacity(case["hi"], 1, max(k, 1))
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 31 + 5)
    s.eng = eng = Engine(m.cfg(), B, cap, k)
    tw, dw = _weights(m, k, seed, kind == "draft")
    eng.bind(tw, dw if k > 0 else None)
    if kind == "prefill":
        s.prompts = [synth.rng(seed, 901 + i).integers(0, m.vocab, size=n).astype("int32") for i, n in enumerate(lens)]
        return s
    # committed prefixes: K and V rows of order one, as the models' own projections give
    plain = torch.empty(B, m.n_kv_heads, cap, m.head_dim, dtype=eng.tdtype, device="cuda")
    for which, layer in [(w, l) for w in ("tk", "tv") for l in range(m.n_layers)] + [("dk", 0), ("dv", 0)]:
        if which[0] == "t" and kind == "draft" or which[0] == "d" and k == 0:
            continue
        eng.sf_kv_import(plain.normal_(generator=g), which, layer)
    del plain
    # the step before this one committed n_new tokens: their hooked states are in hand, newest last
    pending = _uniform((B,), 0, m.vocab, g)
    n_new = torch.minimum(_uniform((B,), 1, k + 2, g), torch.tensor(lens, dtype=torch.int32, device="cuda"))
    row = torch.arange(k + 1, device="cuda")[None, :]
    token = (pending[:, None].long() - n_new[:, None].long() + row) % m.vocab
    hooks = tw["embed"][token][:, :, None, :] + torch.randn(B, k + 1, 4, m.d_model, generator=g, device="cuda") * 4.0
    s.hooks = hooks.to(eng.tdtype)
    slot = torch.arange(1, k + 1, device="cuda")[None, :]
    wrong = torch.rand(B, k, generator=g, device="cuda") > ACCEPT_PROB
    s.guess = ((pending[:, None].long() + slot + 7 * wrong) % m.vocab).to(torch.int32)
    eng.set_state(kv_len=lens, pending=pending.cpu().numpy(), n_new=n_new.cpu().numpy())
    eng.hooks.copy_(s.hooks)
    s.ints = [eng.kv_len.clone(), eng.pending.clone(), eng.n_new.clone()]
    s.len_upper = eng.len_upper
    i32 = dict(dtype=torch.int32, device="cuda")
    s.draft, s.ids, s.tokens = torch.empty(B, k, **i32), torch.empty(B, k + 1, **i32), torch.empty(B, k + 1, **i32)
    s.accepted = torch.empty(B, **i32)
    q = k if kind == "draft" else k + 1
    s.logits = torch.empty(B, q, m.vocab, dtype=torch.float32, device="cuda") if case["logits"] else None
    s.graph = None
    if case["graph"]:
        # a serving loop records its step once and replays it
        eng.pin_len_upper()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _decode(s)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s.graph):
            _decode(s)
        torch.cuda.synchronize()
    return s


def _decode(s):
    eng, k = s.eng, s.k
    if k > 0:
        eng.sf_draft_step(k, mask=s.mask, draft_out=s.draft)
    eng.sf_verify_step(k, s.guess, logits_out=s.logits, ids_out=s.ids, logits=s.logits is not None)
    eng.sf_accept_commit(k, s.guess, s.ids, accept_out=s.accepted, tokens_out=s.tokens)


def run(s):
    eng, kind = s.eng, s.case["kind"]
    if kind == "prefill":
        first = eng.prefill(s.prompts, block=s.case["block"])
        return {"first": first, "kv_len": eng.kv_len, "pending": eng.pending, "hooks": eng.hooks, "n_new": eng.n_new,
                "tk": eng.layer_cache("tk", eng.L - 1), "tv": eng.layer_cache("tv", eng.L - 1), "dk": eng.dk, "dv": eng.dv}
    if kind == "draft":
        eng.sf_draft_step(s.k, mask=s.mask, draft_out=s.draft, logits_out=s.logits)
        return {"draft": s.draft, "logits": s.logits, "dk": eng.dk, "dv": eng.dv}
    # the same point of the generation in every pass: committed lengths, pending tokens, newest hooked states
    torch._foreach_copy_([eng.kv_len, eng.pending, eng.n_new], s.ints)
    eng.hooks.copy_(s.hooks)
    if s.graph is not None:
        s.graph.replay()
    else:
        eng.len_upper = s.len_upper
        _decode(s)
    out = {"ids": s.ids, "accepted": s.accepted, "tokens": s.tokens, "kv_len": eng.kv_len, "pending": eng.pending,
           "n_new": eng.n_new, "cu_new": eng.cu_new, "hooks": eng.hooks, "tk": eng.layer_cache("tk", eng.L - 1),
           "tv": eng.layer_cache("tv", eng.L - 1)}
    if s.k > 0:
        out.update(draft=s.draft, dk=eng.dk, dv=eng.dv)
    if s.logits is not None:
        out["logits"] = s.logits
    return out


def _pass_work(m, rows, keys, scored, wants_logits):
    """Target forward of `rows` rows whose attention reads `keys` cached positions once and scores `scored`
    (row, key) pairs: weights once, caches once, embedding rows in, hooked states (and logits) out."""
    es = 2 if m.dtype == "bf16" else 4
    d, F, nq, nkv = m.d_model, m.d_ffn, m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    per_layer = d * (nq + 2 * nkv) + nq * d + 3 * d * F
    by = m.n_layers * (per_layer + 2 * nkv * (keys + rows)) * es + m.vocab * d * es + rows * d * es * 5
    fl = m.n_layers * (2.0 * rows * per_layer + 4.0 * nq * scored) + 2.0 * rows * m.vocab * d
    return by + (rows * m.vocab * 4 if wants_logits else 0), fl


def _draft_work(m, B, k, keys, two_stage, wants_logits):
    es = 2 if m.dtype == "bf16" else 4
    d, F, nq, nkv = m.d_model, m.d_ffn, m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    layer = d * (nq + 2 * nkv) + nq * d + 3 * d * F
    rows, new = B * k, B * (k + 1)
    extra = d * (nq + 2 * nkv) + nq * d if two_stage else 0
    by = (4 * d * d + k * d * d + layer + extra + m.vocab * d + 2 * nkv * keys + new * 4 * d) * es
    fl = 2.0 * new * (4 * d * d + 2 * d * nkv) + 2.0 * B * k * d * d + 2.0 * rows * layer + 2.0 * rows * m.vocab * d
    fl += 2.0 * B * extra + 4.0 * nq * keys * (1 if two_stage else k)
    return by + (rows * m.vocab * 4 if wants_logits else 0), fl


def work(case):
    m, B, k = _shape(case), case["batch"], case["k"]
    n = (case["lo"] + case["hi"]) / 2.0
    if case["kind"] == "prefill":
        tok = B * n
        by, fl = _pass_work(m, tok, 0, tok * n / 2, False)
        fl -= 2.0 * (tok - B) * m.vocab * m.d_model       # one choice per prompt is needed, not one per token
        es = 2 if m.dtype == "bf16" else 4
        nkv = m.n_kv_heads * m.head_dim
        by += (4 * m.d_model + 2 * nkv) * m.d_model * es + tok * 2 * nkv * es
        fl += 2.0 * tok * (4 * m.d_model + 2 * nkv) * m.d_model
        return {"bytes": by, "flops": fl}
    if case["kind"] == "draft":
        by, fl = _draft_work(m, B, k, B * n, True, case["logits"])
        return {"bytes": by, "flops": fl}
    by, fl = _pass_work(m, B * (k + 1), B * n, B * (k + 1) * n, case["logits"])
    if k > 0:
        b2, f2 = _draft_work(m, B, k, B * n, False, False)
        by, fl = by + b2, fl + f2
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """bf16: the same passes with the linear layers' K range split otherwise and the attention's keys cut otherwise
    move logits and hooked states by up to 3.0e-3 (2-norm) and single K/V values by up to 2.8e-2 of themselves, and
    no token; four times that is allowed.  fp32: other orders of the 256- to 1024-term sums."""
    if case["model"] == "tiny":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.002}
    return {"rel": 1.2e-2, "max": 0.11, "differ": 0.002}
