"""The workloads whose speed this framework is judged by: what a user has it do, through `Session` and `fit_scores`.

Five kinds of call, over the model shapes of the repository's configurations and small generic ones:

* `step`      a stretch of speculative decoding on a running sequence: `steps` times draft, verify, accept, rollback, and
              after each the read-back that tells the program which tokens it got;
* `plain`     the same stretch with plain autoregressive decoding, the thing speculation is compared with;
* `prefill`   a prompt's forward: fills the cache, yields the first token;
* `generate`  the whole outer loop (`Session.generate`): prompt, then tokens until the wanted number is there;
* `fit`       the draft's construction: layer scores of a calibration set.

The weights are random, but laid out so that the next-token distributions look like a trained model's and not like
noise: every token has a likely successor (and, for sampling, a second one that is drawn now and then), so that drafts are
accepted, and the layers contribute about as much to the residual stream as the embedding does.  Greedy choices are then
not near-ties, which a last-bit difference between two correct implementations would decide.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2602_05499_amd as P
from paper_2602_05499_amd.session import fit_scores

DEVICE = "cuda:0"

# widths of the model shapes: full depth, d_model, heads, KV heads, head_dim, d_ffn, vocab, rope theta
SHAPES = {
    "tiny": (4, 256, 4, 4, 64, 688, 1024, 1e4),            # float32 configuration of the test-suite
    "small": (8, 1024, 16, 4, 64, 2816, 32000, 1e4),       # generic small grouped-query model
    "narrow": (6, 512, 16, 8, 32, 1376, 8192, 1e4),        # generic, head_dim 32
    "7b": (32, 4096, 32, 32, 128, 11008, 32000, 1e4),
    "13b": (40, 5120, 40, 40, 128, 13824, 32000, 1e4),
    "l3-8b": (32, 4096, 32, 8, 128, 14336, 128256, 5e5),
    "70b": (80, 8192, 64, 8, 128, 28672, 32000, 1e4),
}


def _case(kind, shape, **kw):
    c = {"kind": kind, "shape": shape, "layers": SHAPES[shape][0], "dtype": "bf16", "mode": "greedy", "K": 4, "prompt": 512,
         "steps": 1, "gen": 0, "samples": 0, "skip": 0.5}
    c.update(kw)
    return c


def listed():
    cases = {
        # one step of the float32 configuration the test-suite is built on: a few hundred microseconds, all latency
        "tiny-step": _case("step", "tiny", dtype="f32", prompt=32),
        # a whole short chat turn on a small model with sampling, ragged sizes: launches, host loop and read-backs count
        "small-generate": _case("generate", "small", mode="sample", K=3, prompt=77, gen=33),
        # the headline workload: greedy speculation on the 7B shape
        "7b-step": _case("step", "7b", prompt=512, steps=4),
        # its baseline, and what a program without a draft runs: one token per forward, at an odd context
        "7b-plain": _case("plain", "7b", K=0, prompt=731, steps=6),
        # deeper speculation with rejection sampling, the second workload of the paper's evaluation
        "13b-step-sample": _case("step", "13b", mode="sample", K=6, prompt=1024, steps=2, skip=0.4),
        # long context, grouped-query heads, a large vocabulary: attention-heavy verification
        "l3-8b-step-long": _case("step", "l3-8b", prompt=4001, steps=2, skip=0.375),
        # the widest layers; a tenth of the depth, so that three states fit the card (time goes linearly with depth)
        "70b-widths-step": _case("step", "70b", layers=8, K=5, prompt=1024, steps=4),
        # an ordinary prompt
        "7b-prefill-512": _case("prefill", "7b", prompt=512),
        # a short follow-up prompt of a chat, sampled
        "7b-prefill-37": _case("prefill", "7b", mode="sample", prompt=37),
        # a ragged prompt at widths that are not powers of two
        "13b-prefill-777": _case("prefill", "13b", prompt=777),
        # the longest prompt of the configurations
        "l3-8b-prefill-4096": _case("prefill", "l3-8b", prompt=4096),
        # ranking the layers of the 7B shape before a draft is cut from it
        "7b-fit": _case("fit", "7b", K=0, prompt=512, samples=2),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; sizes spread over their logarithm, odd ones among them."""
    limit = _cost(_case("prefill", "l3-8b", prompt=4096))
    while True:
        kind = rng.choice(["step", "step", "plain", "prefill", "prefill", "generate", "fit"])
        shape = rng.choice(["tiny", "small", "narrow", "7b", "7b", "13b", "l3-8b", "70b"])
        full = SHAPES[shape][0]
        c = _case(kind, shape, skip=rng.choice([0.375, 0.4, 0.5]),
                  mode=rng.choice(["greedy", "greedy", "sample"]), K=rng.randint(1, 8))
        c["layers"] = full if shape in ("tiny", "small", "narrow") else rng.randint(2, min(full, {"70b": 8}.get(shape, full)))
        if shape == "tiny":
            c["dtype"] = "f32" if kind != "fit" else "bf16"
        if kind == "fit":
            # sequences of the calibration set; widths of the FIT pass are multiples of 32
            if shape == "tiny":
                continue
            c.update(mode="greedy", K=0, samples=rng.randint(1, 4), prompt=_log_int(rng, 48, 1024))
        elif kind == "prefill":
            c["prompt"] = _log_int(rng, 3, 4096)
        elif kind == "generate":
            c.update(prompt=_log_int(rng, 8, 1024), gen=_log_int(rng, 8, 64))
        else:
            c.update(prompt=_log_int(rng, 16, 4096), steps=rng.randint(1, 6))
            if kind == "plain":
                c["K"] = 0
        if c["dtype"] == "f32":
            c["prompt"] = min(c["prompt"], 1024)
        if _cost(c) <= limit:
            return c


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def _dims(c):
    return SHAPES[c["shape"]][1:7]


def _layer_params(c):
    d, H, Hk, hd, F, V = _dims(c)
    return (H * hd + 2 * Hk * hd) * d + d * H * hd, 3 * F * d


def _n_active(c):
    return c["layers"] - int(c["skip"] * c["layers"])


def _forward_work(c, layers, rows, ctx):
    """One forward of `rows` rows at `ctx` cached positions: every weight and cached row read once."""
    d, H, Hk, hd, F, V = _dims(c)
    B = 4 if c["dtype"] == "f32" else 2
    attn, ffn = _layer_params(c)
    by = layers * ((attn + ffn) * B + 2 * Hk * hd * B * (ctx + rows)) + V * d * B + rows * V * 4
    fl = 2 * rows * (layers * (attn + ffn) + V * d) + layers * 4 * rows * ctx * H * hd
    return by, fl


def _prompt_work(c, n):
    d, H, Hk, hd, F, V = _dims(c)
    B = 4 if c["dtype"] == "f32" else 2
    attn, ffn = _layer_params(c)
    by = c["layers"] * ((attn + ffn) * B + 2 * Hk * hd * B * n) + V * d * B + n * d * B
    fl = 2 * (c["layers"] * (n * (attn + ffn) + H * hd * n * (n + 1)) + V * d)
    return by, fl


def _step_work(c, ctx):
    drafts = [_forward_work(c, _n_active(c), 1, ctx + i) for i in range(c["K"])]
    v = _forward_work(c, c["layers"], c["K"] + 1, ctx + c["K"])
    return v[0] + sum(b for b, _ in drafts), v[1] + sum(f for _, f in drafts)


def work(case):
    c = case
    by = fl = 0
    if c["kind"] in ("prefill", "generate"):
        by, fl = _prompt_work(c, c["prompt"])
    n = c["steps"] if c["kind"] in ("step", "plain") else 0
    if c["kind"] == "generate":
        n = -(-(c["gen"] - 1) // (c["K"] + 1))      # every draft accepted
    for i in range(n):
        b, f = _step_work(c, c["prompt"] + i * (c["K"] + 1))
        by, fl = by + b, fl + f
    if c["kind"] == "fit":
        d, H, Hk, hd, F, V = _dims(c)
        attn, ffn = _layer_params(c)
        T, L = c["prompt"], c["layers"]
        # forward and backward-data products, causal attention (two products forward, four backward), and per matrix the
        # Gram matrix of its output gradient, per distinct input that of the input: symmetric, half of each
        per = 4 * T * (L * (attn + ffn) + V * d) + L * 6 * T * T * H * hd
        per += L * T * T * ((H * hd + 2 * Hk * hd + d + 2 * F + d) + (d + H * hd + d + F))
        by, fl = (L * (attn + ffn) + V * d) * 2, per * c["samples"]
    return {"bytes": by, "flops": fl}


def _cost(c):
    """A rough time, to keep drawn cases below the largest listed one."""
    w = work(c)
    rate = 2e13 if c["dtype"] == "f32" else (1.5e14 if c["kind"] == "fit" else 3e14)
    return w["bytes"] / 5e12 + w["flops"] / rate


def tolerance(case):
    # Measured against the same prompt forward in torch (sums in another order), 2-norm over 2-norm: float32 storage 1e-6
    # of the logits and of the cache; bfloat16 storage 2-7e-4 of the logits and up to 1.3e-3 of the cache at 32 layers
    # (keys and values are rounded when they enter it, a few round the other way after a last-bit difference, and the
    # layers behind amplify that).  FIT scores: float32 sums of about a million terms in another order, 1-4e-7 against a
    # float64 evaluation.  About four times these.
    if case["kind"] == "fit":
        return {"rel": 2e-6}
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "differ": 0.05}
    return {"rel": 6e-3, "differ": 0.05}


# ---- inputs ----------------------------------------------------------------------------------------------------------
def _shape(c):
    L, d, H, Hk, hd, F, V, theta = SHAPES[c["shape"]]
    return SimpleNamespace(name=c["shape"], n_layers=c["layers"], d_model=d, n_heads=H, n_kv_heads=Hk, head_dim=hd, d_ffn=F,
                           vocab=V, dtype=c["dtype"], rms_eps=1e-5, rope_theta=theta)


def _weights(c, s, gen):
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    d, hq, hk = s.d_model, s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim

    def mat(rows, cols, std):
        return torch.empty(rows, cols, dtype=dt, device=DEVICE).normal_(0.0, std, generator=gen)

    def gain():
        return 1.0 + 0.1 * torch.randn(d, device=DEVICE, generator=gen)

    # per-row input deviation 1 after the norm; the residual branches scaled down with depth, as models are initialised
    g, res = 1.28 / math.sqrt(d), 1.0 / math.sqrt(2.0 * s.n_layers)
    layers = [{"attn_norm": gain(), "wq": mat(hq, d, g), "wk": mat(hk, d, g), "wv": mat(hk, d, g),
               "wo": mat(d, hq, 1.28 / math.sqrt(hq) * res), "ffn_norm": gain(), "w_gate": mat(s.d_ffn, d, g),
               "w_up": mat(s.d_ffn, d, g), "w_down": mat(d, s.d_ffn, 2.0 / math.sqrt(s.d_ffn) * res)}
              for _ in range(s.n_layers)]
    emb = mat(s.vocab, d, 1.0)
    # the successor of token t gets a logit some 20 above the bulk (whose soft-max mass is that of one logit at 11), a
    # second one 3 (sampling) or 10 (greedy: no near-ties) below it
    first, second = (20.0, 17.0) if c["mode"] == "sample" else (20.0, 10.0)
    unit = 1.46 / math.sqrt(d)
    p1 = torch.randperm(s.vocab, device=DEVICE, generator=gen)
    p2 = torch.randperm(s.vocab, device=DEVICE, generator=gen)
    head = mat(s.vocab, d, g)
    blk = 16384
    for r in range(0, s.vocab, blk):
        rows = slice(r, min(s.vocab, r + blk))
        mix = emb[p1[rows]].float() * (first * unit / math.sqrt(d)) + emb[p2[rows]].float() * (second * unit / math.sqrt(d))
        head[rows] += mix.to(dt)
    return SimpleNamespace(tok_emb=emb, final_norm=torch.ones(d, device=DEVICE), lm_head=head, layers=layers)


def prepare(case, seed):
    c = case
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    s = _shape(c)
    w = _weights(c, s, gen)
    if c["kind"] == "fit":
        toks = rng.integers(0, s.vocab, (c["samples"], c["prompt"])).astype(np.int32)
        return SimpleNamespace(case=c, shape=s, weights=w, tokens=toks)
    mask = np.zeros(s.n_layers, np.uint8)          # whole layers: attention and feed-forward bit
    mask[rng.permutation(s.n_layers)[:int(c["skip"] * s.n_layers)]] = 3
    K, n = c["K"], c["prompt"]
    extra = c["steps"] * (K + 1) if c["kind"] in ("step", "plain") else c["gen"]
    st = SimpleNamespace(case=c, mode=P.SD_SAMPLE if c["mode"] == "sample" else P.SD_GREEDY)
    # the list of committed tokens is long enough for many passes: a program that rewinds does not prefill again
    st.ses = P.Session(s, w, mask, max_seq=n + extra + 2 * (K + 1) + 2, max_k=K, max_out=1 << 20, temperature=1.0)
    st.ses.keep_logits(True)                  # logits of every verify row, also when greedy
    st.prompt = rng.integers(0, s.vocab, n).astype(np.int32)
    per = 2 * K + 1
    st.uniforms = rng.random(1 + per * (max(c["steps"], c["gen"]) + 1)).astype(np.float32)
    st.uniforms = np.minimum(st.uniforms, np.float32(1.0 - 2.0 ** -24))
    if c["kind"] in ("step", "plain"):        # the sequence is running: its prompt is in the cache
        st.ses.prefill(st.prompt, st.mode, st.uniforms[:1])
        st.first = st.ses.read(0)[1]["t_last"]
    return st


def _kv(ses):
    return ses.kv.view(torch.float32 if ses.shape.dtype == "f32" else torch.bfloat16)


def _run_stretch(st):
    """`steps` steps from the end of the prompt on; the program reads what each step committed before it goes on."""
    c, ses, K = st.case, st.ses, st.case["K"]
    ses.set_pending(c["prompt"], st.first)
    per, tokens = 2 * K + 1, np.full((c["steps"], K + 1), -1, np.int32)   # a row per step, -1 behind what it committed
    for i in range(c["steps"]):
        u = st.uniforms[1 + i * per:1 + (i + 1) * per] if st.mode == P.SD_SAMPLE else None
        if c["kind"] == "plain":
            ses.decode(st.mode, u)
        else:
            ses.step(K, st.mode, u)
        stats = ses.read(0)[1]
        n = stats["last_n"]
        tokens[i, :n] = ses.dump_draft(K)[:n]
        tokens[i, n] = stats["t_last"]
    return {"tokens": tokens, "logits": ses.dump_logits(P.SD_LOGITS_VERIFY, K + 1), "kv": _kv(ses)}


def run(state):
    c = state.case
    if c["kind"] == "fit":
        ta, tf, losses = fit_scores(state.shape, state.weights, state.tokens)
        return {"attn": ta, "ffn": tf, "loss": losses}
    if c["kind"] in ("step", "plain"):
        return _run_stretch(state)
    ses = state.ses
    if c["kind"] == "prefill":
        ses.prefill(state.prompt, state.mode, state.uniforms[:1])
        first = ses.read(0)[1]["t_last"]
        return {"token": int(first), "logits": ses.dump_logits(P.SD_LOGITS_VERIFY, 1), "kv": _kv(ses)}
    toks, stats = ses.generate(state.prompt, c["gen"], c["K"], state.mode, state.uniforms)
    return {"tokens": toks, "logits": ses.dump_logits(P.SD_LOGITS_VERIFY, c["K"] + 1), "kv": _kv(ses)}
