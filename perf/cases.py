"""What a program does with this library, as timed cases: prompts to their first token, prompts with
generated tokens behind them, and batches of sequences in lock step.

The library holds one model at a time, so the session (weights, workspace, captured graphs, and the page
pool of a batch) is what such a program keeps between calls; it is kept here per model shape and opened
again when a case of another shape comes.  The inputs of a case are its prompts, drawn from the seed.

Models: the 2-layer toy decoder and the LLaMA-2-7B shape of ``workloads.py``, the latter whole or with
1, 2 or 4 of its layers and a vocabulary of 1024, so that single layers are what is timed and compared.
Matrices are N(0, 0.02^2).  A trained model's choice among tokens is clear where i.i.d. matrices would
leave near ties: row perm[t] of the LM head is a multiple of embedding row t and the embedding is large
enough for the residual stream to keep a share of it, so that the next token is perm[t] by a wide margin
while most of every logit still comes out of the layers.
"""
import math
import random

import numpy as np
import torch

from paper_2604_23467_amd import binding, workloads

DEVICE = "cuda:0"
MATRIX_STD = 0.02
WEIGHT_SEED = 7
SAMPLING = dict(temperature=0.8, top_k=50, top_p=0.95)
PAGE_TOKENS = 16
# prompt lengths of a mixed batch, repeated over its sequences (the lengths of the latency protocol)
BATCH_PROMPTS = (10, 25, 50, 100, 250, 500)


def _case(name, kind, model, layers, prompt, new=0, batch=0, sampled=False, lean=False):
    return dict(name=name, kind=kind, model=model, layers=layers, prompt=prompt, new=new, batch=batch,
                sampled=sampled, lean=lean)


def listed():
    return [
        # a toy model's whole request: launches and host calls are what it costs
        _case("tiny answer 10+16", "generate", "tiny", 2, 10, new=16),
        # time to first token of the whole 7B model: the shortest and the longest prompt of the protocol
        _case("7b first token 10", "prefill", "7b", 32, 10),
        _case("7b first token 500", "prefill", "7b", 32, 500),
        # a chat turn of the whole model: short prompt, greedy answer
        _case("7b answer 25+32", "generate", "7b", 32, 25, new=32),
        # layers of the 7B shape under the protocol's other prompt lengths; 350 fills no power of two
        _case("layers first token 50", "prefill", "7b", 4, 50),
        _case("layers first token 100", "prefill", "7b", 4, 100),
        _case("layers first token 250", "prefill", "7b", 4, 250),
        _case("layers first token 350", "prefill", "7b", 4, 350),
        # a prompt of at most 32 tokens from a program that may not allocate
        _case("layers static 25", "static", "7b", 4, 25),
        # a long document and a sampled answer: chunked prefill, decode attention over a long cache
        _case("layers answer 2000+32", "generate", "7b", 4, 2000, new=32, sampled=True),
        # serving: sequences of mixed lengths join, advance together over a paged cache, and leave
        _case("layers batch 16+64", "batch", "7b", 4, 500, new=64, batch=16),
        _case("layers batch 32+64", "batch", "7b", 4, 500, new=64, batch=32, sampled=True),
    ]


def draw(rng):
    """A case of the same ranges: any prompt length up to 2000, any number of layers up to 4."""
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(("prefill", "prefill", "prefill", "generate", "generate", "batch", "static"))
    model = rng.choice(("tiny", "7b", "7b", "7b"))
    layers = 2 if model == "tiny" else rng.choice((1, 2, 4))
    new = batch = 0
    sampled = lean = False
    if kind == "prefill":
        prompt = log_int(1, 2000)
        lean = rng.random() < 0.2
    elif kind == "static":
        prompt = rng.randint(1, 32)
    elif kind == "generate":
        prompt, new, sampled = log_int(1, 2000), log_int(1, 64), rng.random() < 0.5
    else:
        prompt, new, batch, sampled = log_int(10, 500), log_int(4, 64), rng.randint(1, 32), rng.random() < 0.5
    c = _case("", kind, model, layers, prompt, new, batch, sampled, lean)
    del c["name"]
    return c


def _shape(case):
    max_seq = 1024 if case["prompt"] + case["new"] < 1024 else 4096
    if case["model"] == "tiny":
        return workloads.tiny_cfg(max_seq=max_seq)
    whole = workloads.llama7b_cfg(max_seq=max_seq)
    if case["layers"] == whole["n_layers"]:
        return whole
    return workloads.llama7b_cfg(n_layers=case["layers"], vocab=1024, max_seq=max_seq)


def _weights(cfg):
    """(weights, perm): fp16 tensors on the GPU; the LM head's row perm[t] points along embedding row t."""
    d, F, V, L = cfg["d_model"], cfg["ffn_hidden"], cfg["vocab"], cfg["n_layers"]
    g = torch.Generator(device=DEVICE)
    g.manual_seed(WEIGHT_SEED)

    def matrix(rows, cols, std=MATRIX_STD):
        return torch.empty(rows, cols, dtype=torch.float16, device=DEVICE).normal_(0.0, std, generator=g)

    def gain():
        return torch.empty(d, dtype=torch.float16, device=DEVICE).normal_(1.0, 0.1, generator=g)

    # what one layer adds to an element of the residual stream, roughly, and the share of the final
    # stream that is to be left of the embedding: enough to stand out of V random logits
    g1 = MATRIX_STD * math.sqrt(d)
    added = math.sqrt(L) * math.hypot(0.5 * g1 * g1, 0.6 * g1 * g1 * MATRIX_STD * math.sqrt(F) * 0.75)
    share = min(0.6, max(0.25, 9.0 / math.sqrt(d)))
    emb_std = added * share / math.sqrt(1.0 - share * share)
    w = dict(tok_emb=matrix(V, d, emb_std))
    perm = torch.randperm(V, generator=g, device=DEVICE)
    head_std = MATRIX_STD * 64.0 / math.sqrt(d)           # logits of one size whatever the width
    head = torch.empty(V, d, dtype=torch.float16, device=DEVICE)
    head[perm] = (w["tok_emb"].float() * (head_std / emb_std)).half()
    w.update(lm_head=head, final_norm=gain())
    w["layers"] = [dict(attn_norm=gain(), wq=matrix(d, d), wk=matrix(d, d), wv=matrix(d, d), wo=matrix(d, d),
                        ffn_norm=gain(), w_gate=matrix(F, d), w_up=matrix(F, d), w_down=matrix(d, F))
                   for _ in range(L)]
    return w, perm


_open = {}            # the one open session: key, session, weights, perm


def _model(case):
    """The weights of the case's model, made again only when the shape changes."""
    key = tuple(sorted(_shape(case).items()))
    if _open.get("weights_key") != key:
        _close()
        _open["weights"], _open["perm"] = _weights(_shape(case))
        _open["weights_key"] = key
    return _open["weights"], _open["perm"]


def _close():
    if "session" in _open:
        _open["session"].close()
    _open.clear()
    if torch.cuda.is_available():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()


def _batch_prompts(case):
    return [min(case["prompt"], BATCH_PROMPTS[i % len(BATCH_PROMPTS)]) for i in range(case["batch"])]


def _pages(case):
    return 1 + sum(-(-(n + case["new"] + 1) // PAGE_TOKENS) for n in _batch_prompts(case))


def _session(case):
    key = (tuple(sorted(_shape(case).items())), case["lean"], case["sampled"],
           (case["batch"], _pages(case)) if case["batch"] else None)
    if _open.get("key") != key:
        if "session" in _open:
            _open.pop("session").close()
            _open.pop("key", None)
        weights, _ = _model(case)
        s = binding.Session(_shape(case), weights, flags=binding.LL_FLAG_LEAN_WORKSPACE if case["lean"] else 0)
        if case["batch"]:
            s.ll_batch_open(case["batch"], PAGE_TOKENS, _pages(case))
        if case["sampled"]:
            s.ll_set_sampling(seed=11, **SAMPLING)
        _open["session"], _open["key"] = s, key
    return _open["session"]


def _prompts(case, seed):
    rng = random.Random(seed)
    lengths = _batch_prompts(case) if case["batch"] else [case["prompt"]]
    vocab = _shape(case)["vocab"]
    return [np.array([rng.randrange(vocab) for _ in range(n)], dtype=np.int32) for n in lengths]


def prepare(case, seed):
    _session(case)
    return dict(case=case, prompts=_prompts(case, seed))


def run(state):
    case = state["case"]
    s = _session(case)
    if case["kind"] == "batch":
        slots, first = [], []
        for p in state["prompts"]:
            slot, token = s.ll_batch_add(p)
            slots.append(slot)
            first.append(token)
        steps = [s.ll_batch_step() for _ in range(case["new"])]
        logits = np.stack([s.ll_batch_dbg_get_logits(i) for i in slots])
        for i in slots:
            s.ll_batch_remove(i)
        tokens = np.array([[first[j]] + [row[i] for row in steps] for j, i in enumerate(slots)])
        return dict(logits=logits, tokens=tokens)
    s.ll_reset()
    first = (s.ll_prefill_static if case["kind"] == "static" else s.ll_prefill)(state["prompts"][0])
    tokens = [first]
    if case["new"]:
        tokens += list(s.ll_decode_n(case["new"]))
    return dict(logits=s.ll_dbg_get_logits(), tokens=np.array(tokens))


def work(case):
    """Every weight once per call of the library, every key and value row read once per step; the
    multiply-adds of each token and of causal attention."""
    cfg = _shape(case)
    d, F, V, L = cfg["d_model"], cfg["ffn_hidden"], cfg["vocab"], cfg["n_layers"]
    layers = L * (4 * d * d + 3 * d * F)
    passes, rows = 0, 0
    nbytes = flops = 0.0
    lengths = _batch_prompts(case) if case["batch"] else [case["prompt"]]
    for n in lengths:                                    # prefill: the weights, the new K/V rows, one row of logits
        passes += 1
        rows += n
        nbytes += 2 * L * 2 * d * n
        flops += 2.0 * layers * n + 2.0 * V * d + L * 2.0 * d * n * (n + 1)
    passes += case["new"]
    for i in range(case["new"]):                         # decode steps: all sequences of a batch share the weights
        for n in lengths:
            nbytes += 2 * L * 2 * d * (n + i + 1)
            flops += 2.0 * (layers + V * d) + L * 4.0 * d * (n + i + 1)
    nbytes += passes * 2.0 * (layers + V * d) + 2.0 * d * rows
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    # fp16 weights, cache and matrix operands: measured against fp64 0.0008 .. 0.0012 over one to four layers and
    # 0.0011 .. 0.0020 where the logits travel through 32; four times that
    return dict(rel=0.008 if case["layers"] == 32 else 0.005, differ=0.002)


def _forward(cfg, w, tokens, first):
    """Logits (fp64) of positions first .. of one sequence: the decoder as plain matrix products."""
    d, H, hd = cfg["d_model"], cfg["n_heads"], cfg["head_dim"]
    n, hh = len(tokens), hd // 2
    f = lambda t: t.double()
    x = f(w["tok_emb"][torch.as_tensor(np.asarray(tokens, dtype=np.int64), device=DEVICE)])
    pos = torch.arange(n, dtype=torch.float64, device=DEVICE)
    freq = cfg["rope_theta"] ** (-2.0 * torch.arange(hh, dtype=torch.float64, device=DEVICE) / hd)
    cos, sin = torch.cos(pos[:, None] * freq), torch.sin(pos[:, None] * freq)
    mask = torch.full((n, n), -math.inf, dtype=torch.float64, device=DEVICE).triu(1)

    def norm(v, gain):
        return v / torch.sqrt(v.square().mean(-1, keepdim=True) + cfg["rms_eps"]) * f(gain)

    def rotate(v):                                        # [H, n, hd], pairs (j, j + hd / 2)
        a, b = v[..., :hh], v[..., hh:]
        return torch.cat((a * cos - b * sin, b * cos + a * sin), -1).contiguous()

    def heads(v):
        return v.view(n, H, hd).transpose(0, 1).contiguous()

    for lw in w["layers"]:
        h = norm(x, lw["attn_norm"])
        q, k, v = (heads(h @ f(lw[m]).t()) for m in ("wq", "wk", "wv"))
        q, k = rotate(q), rotate(k)
        o = torch.empty_like(q)
        for i in range(H):
            o[i] = torch.softmax(q[i] @ k[i].t() / math.sqrt(hd) + mask, -1) @ v[i]
        x = x + o.transpose(0, 1).reshape(n, d) @ f(lw["wo"]).t()
        h = norm(x, lw["ffn_norm"])
        x = x + (torch.nn.functional.silu(h @ f(lw["w_gate"]).t()) * (h @ f(lw["w_up"]).t())) @ f(lw["w_down"]).t()
    return norm(x[first:], w["final_norm"]) @ f(w["lm_head"]).t()


def exact(case, seed):
    cfg = _shape(case)
    w, perm = _model(case)
    perm = perm.cpu().numpy()
    logits, tokens = [], []
    for p in _prompts(case, seed):
        chain = []                                        # the tokens the model is built to choose
        for _ in range(case["new"]):
            chain.append(int(perm[chain[-1] if chain else p[-1]]))
        for _ in range(8):                                # ... corrected where it chooses others
            rows = _forward(cfg, w, list(p) + chain, len(p) - 1)
            best = [int(t) for t in rows.argmax(-1)]
            if case["sampled"] or best[:-1] == chain:
                break
            at = next(i for i, t in enumerate(chain) if t != best[i])
            chain = best[:at + 1] + [best[at + 1]] * (len(chain) - at - 1)
        logits.append(rows[-1].cpu().numpy())
        tokens.append(best)
    if not case["batch"]:
        logits, tokens = logits[0], tokens[0]
    return dict(logits=np.array(logits), tokens=None if case["sampled"] else np.array(tokens))
