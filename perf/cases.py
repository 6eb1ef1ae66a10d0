"""The work a user of this library has it do, as cases that can be timed.

A case is one pass through the public entry points of ``paper_2608_19889_amd``
(``Model.prefill``, ``decode_step``, ``step`` and ``loss_and_grads``): a greedy
or sampled ``generate`` (kind "generate"), a prompt's prefill alone
("prefill"), the logits of every position ("score"), a continuous-batching run
("serve") or a training step's loss and gradients ("train").  The model shapes
are those of ``synthetic.MODEL_SHAPES`` at full width and vocabulary; most cases
keep only a few layers, so that a layer's rounding is compared and not what a
deep stack makes of it.  Weights are drawn as ``synthetic`` draws them.

Decode tokens are given (as a sampler would hand them over) rather than taken
from the previous argmax, so that one near-tie does not change everything after
it; they are copied into one fixed token buffer per step.
"""
import math
import random
import zlib

import torch

from paper_2608_19889_amd import Model
from synthetic import MODEL_SHAPES, weight_shapes

DEV = "cuda"
PAGE = 16


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest calls: a float32 135M-shaped model, one chat turn of a
        # single user; latency and launches count
        dict(name="f32_135m_b1", kind="generate", model="135m", layers=6, batch=1, lo=32, hi=32, steps=8),
        # the headline workload: 1B-shaped, 8 prompts of 512, the whole model
        dict(name="generate_1b_b8", kind="generate", model="1b", layers=16, batch=8, lo=512, hi=512, steps=64),
        # 7B-shaped decode at batch 16 behind 1k-token prompts
        dict(name="generate_7b_b16", kind="generate", model="7b", layers=4, batch=16, lo=1024, hi=1024, steps=96),
        # offline batch generation: more sequences than one fused decode projection takes
        dict(name="generate_1b_b160", kind="generate", model="1b", layers=4, batch=160, lo=40, hi=88, steps=32),
        # GPT-2 XL-shaped: LayerNorm, learned positions, biases, odd vocabulary
        dict(name="generate_gpt2xl_b8", kind="generate", model="gpt2xl", layers=6, batch=8, lo=384, hi=512, steps=48),
        # mixture of experts: prefill through the grouped GEMM, decode through the grouped projection
        dict(name="generate_moe16b_b32", kind="generate", model="moe16b", layers=3, batch=32, lo=256, hi=256, steps=32),
        # time to first token of one chat turn
        dict(name="prefill_1b_short", kind="prefill", model="1b", layers=4, batch=1, lo=93, hi=93),
        # a full prefill batch of long ragged prompts
        dict(name="prefill_7b_long", kind="prefill", model="7b", layers=2, batch=9, lo=1500, hi=2048),
        # log-likelihood scoring: the logits of every position
        dict(name="score_1b", kind="score", model="1b", layers=2, batch=3, lo=180, hi=400),
        # continuous batching over a paged cache: prompt chunks share steps with decode tokens
        dict(name="serve_7b_paged", kind="serve", model="7b", layers=2, batch=40, lo=64, hi=700, steps=24,
             budget=2048),
        # a training step of the 1B shape, 8 x 512 tokens (tied head)
        dict(name="train_1b", kind="train", model="1b", layers=4, batch=8, lo=512, hi=512),
        # a training step of the 7B shape: biases, untied head, ragged sequences, head dimension 128
        dict(name="train_7b_ragged", kind="train", model="7b", layers=2, batch=5, lo=100, hi=900),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: batches, lengths and step counts
    spread over what each kind is used for, odd values among them."""
    kind = rng.choice(["generate", "generate", "generate", "prefill", "prefill", "score", "serve", "train"])
    if kind == "generate":
        model = rng.choice(["135m", "1b", "1b", "7b", "gpt2xl", "moe16b", "mistral7b"])
        if model == "135m":
            lo = _log_int(rng, 5, 200)
            return dict(kind=kind, model=model, layers=rng.randint(2, 6), batch=rng.randint(1, 6), lo=lo,
                        hi=lo + rng.randint(0, 40), steps=rng.randint(3, 12))
        batch = _log_int(rng, 1, 200 if model != "moe16b" else 64)
        lo = _log_int(rng, 16, max(17, min(700, 12000 // batch)))
        return dict(kind=kind, model=model, layers=rng.randint(2, 3), batch=batch, lo=lo,
                    hi=lo + rng.randint(0, lo // 2), steps=rng.randint(16, 64))
    if kind == "prefill":
        model = rng.choice(["1b", "1b", "7b", "mistral7b", "32b", "gpt2xl"])
        tokens = _log_int(rng, 20, 12000 if model != "gpt2xl" else 4000)
        batch = rng.randint(1, max(1, min(12, tokens // 16)))
        hi = max(2, min(tokens // batch, 1000 if model == "gpt2xl" else 6000))
        return dict(kind=kind, model=model, layers=rng.randint(1, 2), batch=batch, lo=max(1, hi // 2), hi=hi)
    if kind == "score":
        hi = _log_int(rng, 30, 500)
        return dict(kind=kind, model=rng.choice(["1b", "7b"]), layers=rng.randint(1, 2), batch=rng.randint(1, 3),
                    lo=max(2, hi // 2), hi=hi)
    if kind == "serve":
        return dict(kind=kind, model=rng.choice(["1b", "7b"]), layers=2, batch=rng.randint(6, 60),
                    lo=rng.randint(20, 100), hi=rng.randint(200, 800), steps=rng.randint(10, 24),
                    budget=rng.choice([512, 1024, 2048]))
    model = rng.choice(["1b", "7b"])
    hi = _log_int(rng, 64, 1000)
    return dict(kind=kind, model=model, layers=1 if model == "7b" else rng.randint(1, 2),
                batch=max(1, min(8, (3500 if model == "1b" else 2200) // hi)), lo=max(2, hi // 2), hi=hi)


# ------------------------------------------------------------------ inputs

def _shape(case):
    s = dict(MODEL_SHAPES[case["model"]])
    s["num_hidden_layers"] = case["layers"]
    return s


def _lens(case):
    """The prompt lengths: part of the case, not of the seed, so that every
    seed is the same work."""
    r = random.Random("%s %s %s %s" % (case["model"], case["batch"], case["lo"], case["hi"]))
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]


def _weights(shape, seed):
    dt = torch.bfloat16 if shape["dtype"] == "bf16" else torch.float32
    out = {}
    for name, shp in weight_shapes(shape).items():
        g = torch.Generator(device=DEV)
        g.manual_seed((zlib.crc32(name.encode()) ^ (seed << 32)) & ((1 << 63) - 1))
        w = torch.randn(shp, generator=g, device=DEV, dtype=torch.float32).mul_(0.02)
        if name.endswith("layernorm.weight") or name == "model.norm.weight" or (".ln_" in name
                                                                                and name.endswith(".weight")):
            w.add_(1.0)
        out[name] = w.to(dt)
    return out


def _tokens(case, shape, seed):
    """(prompts, one int32 tensor per sequence; decode tokens int32 [steps, batch])"""
    g = torch.Generator(device="cpu")
    g.manual_seed(seed & ((1 << 62) - 1))
    V = shape["vocab_size"]
    seqs = [torch.randint(0, V, (n,), generator=g, dtype=torch.int64).to(torch.int32) for n in _lens(case)]
    dec = torch.randint(0, V, (max(_decode_tokens(case), 1), case["batch"]), generator=g, dtype=torch.int64)
    return seqs, dec.to(torch.int32)


def _plan(case):
    """First-come-first-served schedule of a "serve" case: per step a list of
    (sequence, start, count), count 0 for a decode token.  A step gives every
    running sequence one decode token and fills the rest of the budget with
    prompt chunks in arrival order; the run ends when the last sequence has had
    ``steps`` decode tokens."""
    lens, B = _lens(case), case["batch"]
    fed, dec, plan = [0] * B, [0] * B, []
    while min(dec) < case["steps"]:
        st = [(b, dec[b], 0) for b in range(B) if fed[b] == lens[b]]
        used = len(st)
        for b in range(B):
            c = min(lens[b] - fed[b], case["budget"] - used)
            if c > 0:
                st.append((b, fed[b], c))
                used += c
        for b, _, c in st:
            if c:
                fed[b] += c
            else:
                dec[b] += 1
        plan.append(st)
    return plan


def _decode_tokens(case):
    if case["kind"] == "serve":
        return max(start + 1 for st in _plan(case) for _, start, c in st if c == 0)
    return case.get("steps", 0)


def prepare(case, seed):
    shape = _shape(case)
    V, B, kind = shape["vocab_size"], case["batch"], case["kind"]
    seqs, dec = _tokens(case, shape, seed)
    lens = [len(s) for s in seqs]
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    w = _weights(shape, seed)
    st = dict(case=case, cu=cu, flat=torch.cat(seqs).to(DEV))
    # one more position than the last decode token, as a serving program would leave
    room = max(lens) + _decode_tokens(case) + 1
    if kind == "serve":
        plan = _plan(case)
        need = [-(-(n + _decode_tokens(case)) // PAGE) for n in lens]
        g = torch.Generator(device="cpu")
        g.manual_seed((seed + 1) & ((1 << 62) - 1))
        perm = torch.randperm(sum(need), generator=g).to(torch.int32)
        table = torch.full((B, max(need)), -1, dtype=torch.int32)
        at = 0
        for b, nb in enumerate(need):
            table[b, :nb] = perm[at:at + nb]
            at += nb
        steps = []
        for s in plan:
            slots = [b for b, _, _ in s]
            fresh = [1 if c and start == 0 else 0 for _, start, c in s]
            scu = [0]
            for _, _, c in s:
                scu.append(scu[-1] + (c or 1))
            toks = torch.cat([seqs[b][i:i + c] if c else dec[i, b:b + 1] for b, i, c in s]).to(DEV)
            steps.append((slots, fresh, scu, toks, table[slots] if any(fresh) else None))
        most = max(s[2][-1] for s in steps)
        st.update(model=Model(shape, w, max_batch=B, max_seq=room, max_tokens=most, page_size=PAGE,
                              num_pages=sum(need)), steps=steps,
                  tok=torch.empty(most, dtype=torch.int32, device=DEV),
                  cud=torch.empty(B + 1, dtype=torch.int32, device=DEV),
                  logits=torch.empty((B, V), dtype=torch.float32, device=DEV),
                  nxt=torch.empty(B, dtype=torch.int32, device=DEV))
        return st
    st["model"] = Model(shape, w, max_batch=B, max_seq=room, max_tokens=cu[-1])
    st["nxt"] = torch.empty(B, dtype=torch.int32, device=DEV)
    if kind == "train":
        tg = torch.cat([torch.cat([s[1:], torch.full((1,), -1, dtype=torch.int32)]) for s in seqs])
        st.update(targets=tg.to(DEV), loss=torch.empty(1, dtype=torch.float32, device=DEV),
                  grads={k: torch.empty(tuple(v.shape), dtype=torch.float32, device=DEV) for k, v in w.items()})
        return st
    rows = cu[-1] if kind == "score" else B
    st["first"] = torch.empty((rows, V), dtype=torch.float32, device=DEV)
    if kind == "generate":
        st.update(dec=dec.to(DEV), tok=torch.empty(B, dtype=torch.int32, device=DEV),
                  logits=torch.empty((B, V), dtype=torch.float32, device=DEV))
    return st


def run(st):
    m, kind = st["model"], st["case"]["kind"]
    if kind == "serve":
        for slots, fresh, cu, toks, rows in st["steps"]:
            n = len(slots)
            tok = st["tok"][:cu[-1]]
            tok.copy_(toks)
            m.step(tok, cu, slots, fresh, block_rows=rows, logits=st["logits"][:n], next_tokens=st["nxt"][:n],
                   cu_device=st["cud"])
        return st["logits"]  # the last step decodes one token of every sequence
    if kind == "train":
        m.loss_and_grads(st["flat"], st["cu"], st["targets"], st["grads"], loss=st["loss"])
        return {"loss": st["loss"], "grads": st["grads"]}
    m.prefill(st["flat"], st["cu"], all_logits=kind == "score", logits=st["first"], next_tokens=st["nxt"])
    if kind != "generate":
        return st["first"]
    for i in range(st["case"]["steps"]):
        st["tok"].copy_(st["dec"][i])
        m.decode_step(st["tok"], logits=st["logits"], next_tokens=st["nxt"])
    return [st["first"], st["logits"]]


# ------------------------------------------------------------------ work

def work(case):
    """Bytes and floating-point operations of one pass: per forward call the
    weights once (of a mixture the experts that uniform routing reaches), keys
    and values of the attended positions, token rows and logits once."""
    s = _shape(case)
    gpt2 = s.get("model_type") == "gpt2"
    esz = 2 if s["dtype"] == "bf16" else 4
    D, L, V, H = s["hidden_size"], s["num_hidden_layers"], s["vocab_size"], s["num_attention_heads"]
    KV, hd, I, W = s["num_key_value_heads"], s["head_dim"], s["intermediate_size"], s.get("sliding_window") or 0
    attn_w = (H + 2 * KV) * hd * D + H * hd * D
    mlp_w = (2 if gpt2 else 3) * D * I
    E, k, Ie = s.get("n_routed_experts") or 0, s.get("num_experts_per_tok") or 0, s.get("moe_intermediate_size") or 0
    shared, dense = (s.get("n_shared_experts") or 0) * Ie, (s.get("first_k_dense_replace") or 0) if E else L
    total = {"bytes": 0.0, "flops": 0.0}

    def forward(spans, head_rows):
        """spans: (first position, tokens) of each sequence of the call"""
        T = sum(n for _, n in spans)
        mats, per_token = L * attn_w + dense * mlp_w, L * attn_w + dense * mlp_w
        if E:
            mats += (L - dense) * (D * E + 3 * D * shared + 3 * D * Ie * E * (1 - (1 - k / E) ** T))
            per_token += (L - dense) * (D * E + 3 * D * shared + 3 * D * Ie * k)
        pairs = keys = 0
        for p, n in spans:
            seen = [min(q + 1, W) if W else q + 1 for q in (p, p + n - 1)]
            pairs += n * (seen[0] + seen[1]) / 2 if not W or p + n <= W else \
                sum(min(q + 1, W) for q in range(p, p + n))
            keys += min(p + n, W + n) if W else p + n
        total["bytes"] += (mats + D * V) * esz + 2 * L * KV * hd * esz * (keys + T) + T * D * esz + head_rows * V * 4
        total["flops"] += 2.0 * T * per_token + 2.0 * head_rows * D * V + 4.0 * L * H * hd * pairs

    lens = _lens(case)
    T = sum(lens)
    if case["kind"] == "serve":
        for st in _plan(case):
            forward([(start, c) if c else (lens[b] + start, 1) for b, start, c in st], len(st))
    elif case["kind"] == "train":
        mats = L * (attn_w + mlp_w) + D * V
        pairs = sum(n * (n + 1) / 2 for n in lens)
        grads = mats + (0 if s["tie_word_embeddings"] else D * V)
        # weights read once, every gradient written once in float32
        total = {"bytes": mats * 2.0 + grads * 4.0 + T * D * 2,
                 "flops": 6.0 * T * mats + 14.0 * L * H * hd * pairs}
    else:
        forward([(0, n) for n in lens], T if case["kind"] == "score" else case["batch"])
        for i in range(case.get("steps", 0)):
            forward([(n + i, 1) for n in lens], case["batch"])
    return total


def tolerance(case):
    """Four times the distance to the float64 forward and backward pass
    (``exact``) that the present path shows, and at most 3%: in the 2-norm the
    float32 logits are off by 3e-7, GPT-2's by 0.44%, those of the other bf16
    shapes by 0.8 to 1.4% on two to four layers and by 1.8% on the 16 of the
    whole 1B model, weight gradients by up to 1.3%.  Single values: about six
    standard deviations of that; gradients of rows with few tokens more."""
    if MODEL_SHAPES[case["model"]]["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    if case["kind"] == "train":
        return {"rel": 0.03, "max": 0.9}
    return {"rel": 0.02 if case["model"] == "gpt2xl" else 0.03, "max": 0.4}


# ------------------------------------------------------------------ 64-bit reference

def _forward64(case, s, w, seqs, rows_of):
    """Logits in float64 of the positions ``rows_of(length)`` of each sequence."""
    D, H, KV, hd = s["hidden_size"], s["num_attention_heads"], s["num_key_value_heads"], s["head_dim"]
    W = s.get("sliding_window") or 0
    gpt2 = s.get("model_type") == "gpt2"
    lens = [len(x) for x in seqs]
    ids = torch.cat(seqs).to(DEV).long()
    pos = torch.cat([torch.arange(n, device=DEV) for n in lens])
    get = lambda n: w[n].double()  # noqa: E731

    def rms(x, g):
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + s["rms_norm_eps"]) * g

    def ln(x, p):
        return torch.nn.functional.layer_norm(x, (D,), get(p + ".weight"), get(p + ".bias"),
                                              s["layer_norm_epsilon"])

    def attend(q, k, v):
        outs, at = [], 0
        for n in lens:
            qq, kk, vv = (t[at:at + n].transpose(0, 1) for t in (q, k, v))
            step = max(1, int(2e9 // (8 * n * n)))  # heads at once: scores of at most about 2 GB
            ii = torch.arange(n, device=DEV)
            hide = ii[None, :] > ii[:, None]
            if W:
                hide = hide | (ii[None, :] <= ii[:, None] - W)
            got = []
            for h in range(0, H, step):
                hs = torch.arange(h, min(H, h + step), device=DEV)
                sc = qq[hs] @ kk[hs // (H // KV)].transpose(1, 2).contiguous() / math.sqrt(hd)
                got.append(torch.softmax(sc.masked_fill(hide, -math.inf), -1) @ vv[hs // (H // KV)])
            outs.append(torch.cat(got).transpose(0, 1).reshape(n, H * hd))
            at += n
        return torch.cat(outs)

    def swiglu(x, p):
        return (torch.nn.functional.silu(x @ get(p + "gate_proj.weight").t()) * (x @ get(p + "up_proj.weight").t())
                ) @ get(p + "down_proj.weight").t()

    def moe(x, p):
        probs = torch.softmax(x @ get(p + "gate.weight").t(), -1)
        top, idx = probs.topk(s["num_experts_per_tok"], -1)
        if s.get("norm_topk_prob"):
            top = top / top.sum(-1, keepdim=True)
        out = swiglu(x, p + "shared_experts.") if s.get("n_shared_experts") else torch.zeros_like(x)
        for e in range(s["n_routed_experts"]):
            t, j = (idx == e).nonzero(as_tuple=True)
            if len(t):
                out = out.index_add(0, t, swiglu(x[t], p + "experts.%d." % e) * top[t, j, None])
        return out

    if gpt2:
        x = get("transformer.wte.weight")[ids] + get("transformer.wpe.weight")[pos]
    else:
        x = get("model.embed_tokens.weight")[ids]
        inv = s["rope_theta"] ** (-torch.arange(0, hd, 2, device=DEV, dtype=torch.float64) / hd)
        ang = torch.cat([pos[:, None] * inv] * 2, -1)[:, None, :]
        cos, sin = ang.cos(), ang.sin()

        def rot(t):
            a, b = t.chunk(2, -1)
            return t * cos + torch.cat([-b, a], -1) * sin
    for i in range(s["num_hidden_layers"]):
        if gpt2:
            p = "transformer.h.%d." % i
            h = ln(x, p + "ln_1") @ get(p + "attn.c_attn.weight") + get(p + "attn.c_attn.bias")
            q, k, v = (t.reshape(-1, H, hd) for t in h.split(D, -1))
            x = x + attend(q, k, v) @ get(p + "attn.c_proj.weight") + get(p + "attn.c_proj.bias")
            h = ln(x, p + "ln_2") @ get(p + "mlp.c_fc.weight") + get(p + "mlp.c_fc.bias")
            h = torch.nn.functional.gelu(h, approximate="tanh")
            x = x + h @ get(p + "mlp.c_proj.weight") + get(p + "mlp.c_proj.bias")
            continue
        p = "model.layers.%d." % i
        h = rms(x, get(p + "input_layernorm.weight"))
        qkv = []
        for c, n in (("q", H), ("k", KV), ("v", KV)):
            t = h @ get(p + "self_attn.%s_proj.weight" % c).t()
            if s["attention_bias"]:
                t = t + get(p + "self_attn.%s_proj.bias" % c)
            qkv.append(t.reshape(-1, n, hd))
        x = x + attend(rot(qkv[0]), rot(qkv[1]), qkv[2]) @ get(p + "self_attn.o_proj.weight").t()
        h = rms(x, get(p + "post_attention_layernorm.weight"))
        if s.get("n_routed_experts") and i >= (s.get("first_k_dense_replace") or 0):
            x = x + moe(h, p + "mlp.")
        else:
            x = x + swiglu(h, p + "mlp.")
    at, rows = 0, []
    for n in lens:
        rows += [at + r for r in rows_of(n)]
        at += n
    x = x[torch.tensor(rows, device=DEV)]
    if gpt2:
        return ln(x, "transformer.ln_f") @ get("transformer.wte.weight").t()
    head = "model.embed_tokens.weight" if s["tie_word_embeddings"] else "lm_head.weight"
    return rms(x, get("model.norm.weight")) @ get(head).t()


def exact(case, seed):
    s = _shape(case)
    w = _weights(s, seed)
    seqs, dec = _tokens(case, s, seed)
    kind = case["kind"]
    if kind == "train":
        p = {k: v.double().requires_grad_(True) for k, v in w.items()}
        logits = _forward64(case, s, p, seqs, range)
        tg = torch.cat([torch.cat([x[1:], torch.full((1,), -1, dtype=torch.int32)]) for x in seqs]).to(DEV).long()
        loss = torch.nn.functional.cross_entropy(logits, tg, ignore_index=-1)
        loss.backward()
        return {"loss": loss.detach().reshape(1), "grads": {k: v.grad for k, v in p.items()}}
    with torch.no_grad():
        if kind == "score":
            return _forward64(case, s, w, seqs, range)
        if kind == "prefill":
            return _forward64(case, s, w, seqs, lambda n: [n - 1])
        if kind == "serve":
            fed = {}
            for st in _plan(case):
                for b, start, c in st:
                    if c == 0:
                        fed[b] = start + 1
            full = [torch.cat([x, dec[:fed[b], b]]) for b, x in enumerate(seqs)]
            last = [b for b, _, _ in _plan(case)[-1]]
            return _forward64(case, s, w, full, lambda n: [n - 1])[torch.tensor(last, device=DEV)]
        K = case["steps"]
        both = _forward64(case, s, w, [torch.cat([x, dec[:K, b]]) for b, x in enumerate(seqs)],
                          lambda n: [n - 1 - K, n - 1])
        return [both[0::2].contiguous(), both[1::2].contiguous()]
