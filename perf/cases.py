"""Workloads by which the speed of the decode step is judged.

A case is one call of the library as a serving program makes it: the handle (with its weights laid
out), the KV cache, the inputs and the output buffers exist before, ``run`` is the call.  Entry
points: ``fleet_decode_step`` (one step), ``fleet_decode_layers`` (a range of layers on an fp32
residual stream), ``fleet_decode_step_paged`` (paged cache), ``fleet_decode_tokens`` (several greedy
steps), ``fleet_decode_step_static`` (working memory in the library's own array).

Fields of a case: ``entry`` (the entry point), ``model`` (``reduced``: hidden 1024, 8 Q / 2 KV heads,
FFN 3072; ``qwen3_8b``: hidden 4096, 32 Q / 8 KV heads, FFN 12288), ``layers``, ``vocab`` (0: no LM
head), ``max_batch`` (what the handle is made for) and ``batch``, ``kv_lo`` .. ``kv_hi`` (cache
lengths before the step, uniform over the sequences; equal: one length), ``capacity`` (cache slots
per sequence), ``page`` (slots per page, 0: contiguous cache), ``tokens`` (greedy steps per call, 0:
one step), ``ids`` (the step starts from token ids instead of hidden states).

Weights are bf16 N(0, 0.02), gains bf16(1 + N(0, 0.02)), hidden states, embedding rows and the cache
bf16 N(0, 1).  Where tokens are generated the head's row t + 1 is the embedding's row t (scaled to
the other weights): a confident next token, as a trained model gives it, so that the sequence of
tokens does not hang on the last bit of a logit.
"""
from __future__ import annotations

import math
import weakref

import torch

import paper_2604_15379_amd as F

MODELS = {
    "reduced": dict(hidden=1024, nq=8, nkv=2, ffn=3072),
    "qwen3_8b": dict(hidden=4096, nq=32, nkv=8, ffn=12288),
}
HD = 128
EPS, THETA = 1e-6, 1e6
QWEN_VOCAB = 151936
PER_LAYER = ("ln1", "wqkv", "q_norm", "k_norm", "wo", "ln2", "wgu", "wdown")


def _case(name, entry, model, layers, vocab, max_batch, batch, kv_lo, kv_hi, capacity, page=0, tokens=0, ids=False):
    return dict(name=name, entry=entry, model=model, layers=layers, vocab=vocab, max_batch=max_batch, batch=batch,
                kv_lo=kv_lo, kv_hi=kv_hi, capacity=capacity, page=page, tokens=tokens, ids=ids)


def listed():
    return [
        # the smallest step: one layer of a small model, one sequence, a short cache -- launch and dependency latency
        _case("small_step_b1", "step", "reduced", 1, 0, 1, 1, 128, 128, 129),
        # a small draft model that writes a few tokens ahead for three sequences of different lengths
        _case("small_tokens_b3", "tokens", "reduced", 2, 2064, 4, 3, 100, 500, 640, tokens=8, ids=True),
        # two layers of the 8B model for one user: a pipeline stage at its lowest batch
        _case("layers2_b1", "step", "qwen3_8b", 2, 0, 1, 1, 1024, 1024, 1025),
        # the head of the model for a few users: token ids in, one layer, final norm and 151936 logits out
        _case("head_b4_ids", "step", "qwen3_8b", 1, QWEN_VOCAB, 4, 4, 512, 512, 1024, ids=True),
        # an odd number of users with very different lengths; working memory in the library's array
        _case("layers2_b5_ragged", "static", "qwen3_8b", 2, 0, 8, 5, 200, 3000, 4096),
        # a pipeline stage on an fp32 residual stream, eight users
        _case("layers2_b8", "layers", "qwen3_8b", 2, 0, 8, 8, 1024, 2048, 2049),
        # a serving batch between two graph sizes on a paged cache
        _case("layers2_b20_paged", "paged", "qwen3_8b", 2, 0, 32, 20, 300, 4000, 4096, page=64),
        # a full serving batch of mixed lengths
        _case("layers2_b32", "step", "qwen3_8b", 2, 0, 32, 32, 1024, 2048, 2049),
        # a large batch of long sequences: cache traffic as large as the weights'
        _case("layer_b64_kv4096", "step", "qwen3_8b", 1, 0, 64, 64, 4096, 4096, 4097),
        # more sequences than one tile of batch rows holds, short and mixed
        _case("layer_b100_short", "step", "qwen3_8b", 1, 0, 128, 100, 100, 1000, 1024),
        # the whole 36-layer model for one user at 1024 tokens
        _case("full_b1", "step", "qwen3_8b", 36, QWEN_VOCAB, 1, 1, 1024, 1024, 1025),
        # the whole model at a full serving batch of mixed lengths
        _case("full_b32", "step", "qwen3_8b", 36, QWEN_VOCAB, 32, 32, 1024, 2048, 2049),
    ]


def draw(rng):
    """One more case of the same ranges: 1 .. 128 sequences, caches of 16 .. 8192 tokens (at most
    262144 in all), one to four layers of either model, with and without the head."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    model = rng.choice(["reduced", "qwen3_8b", "qwen3_8b", "qwen3_8b"])
    batch = log_int(1, 128)
    max_batch = rng.choice([batch, min(128, 1 << (batch - 1).bit_length()), min(128, batch + rng.randint(0, batch))])
    kv_hi = log_int(16, max(17, min(8192, 262144 // batch)))
    kv_lo = kv_hi if rng.random() < 0.3 else rng.randint(max(1, kv_hi // 16), kv_hi)
    entry = rng.choice(["step", "step", "layers", "paged", "static", "tokens"])
    if entry == "static" and max_batch > 16:
        entry = "step"                       # the library's array holds the working memory of up to 16 sequences
    layers = rng.randint(1, 4)
    if batch * kv_hi > 65536:
        layers = 1
    vocab = 0
    if entry == "tokens" or (entry in ("step", "paged") and rng.random() < 0.3):
        vocab = 16 * log_int(60, 1000) if model == "reduced" else 16 * log_int(1000, 9496)
    tokens = rng.randint(2, 12) if entry == "tokens" else 0
    capacity = kv_hi + tokens + rng.choice([1, 1, 63, kv_hi // 2 + 1])
    page = rng.choice([64, 128, 256]) if entry == "paged" else 0
    ids = entry == "tokens" or (vocab > 0 and rng.random() < 0.5)
    c = _case("", entry, model, layers, vocab, max_batch, batch, kv_lo, kv_hi, capacity, page, tokens, ids)
    del c["name"]
    most = work(listed()[-1])["bytes"]
    while work(c)["bytes"] > most:           # fewer steps per call, then fewer layers
        if c["tokens"] > 2:
            c["tokens"] -= 1
        else:
            c["layers"] -= 1
    return c


class _Gen:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, shape, std=1.0, mean=0.0):
        out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        flat = out.view(-1)
        for s in range(0, flat.numel(), 1 << 28):
            n = min(flat.numel() - s, 1 << 28)
            t = torch.randn(n, generator=self.g, device="cuda", dtype=torch.float32)
            flat[s:s + n] = t.mul_(std).add_(mean)
        return out

    def ints(self, lo, hi, n):
        return torch.randint(lo, hi + 1, (n,), generator=self.g, device="cuda", dtype=torch.int32)


def _inputs(case, seed):
    """Weights, cache and inputs of a case, made from the seed alone."""
    m, L, B = MODELS[case["model"]], case["layers"], case["batch"]
    H, nq, nkv, ffn = m["hidden"], m["nq"], m["nkv"], m["ffn"]
    g = _Gen(seed)
    w = {k: [] for k in PER_LAYER}
    for _ in range(L):
        w["ln1"].append(g.normal((H,), 0.02, 1.0))
        w["wqkv"].append(g.normal(((nq + 2 * nkv) * HD, H), 0.02))
        w["q_norm"].append(g.normal((HD,), 0.02, 1.0))
        w["k_norm"].append(g.normal((HD,), 0.02, 1.0))
        w["wo"].append(g.normal((H, nq * HD), 0.02))
        w["ln2"].append(g.normal((H,), 0.02, 1.0))
        w["wgu"].append(g.normal((2 * ffn, H), 0.02))
        w["wdown"].append(g.normal((H, ffn), 0.02))
    V = case["vocab"]
    if V:
        w["final_norm"] = g.normal((H,), 0.02, 1.0)
        if case["ids"]:
            w["embed"] = g.normal((V, H))
        w["lm_head"] = (w["embed"].roll(1, 0) * 0.02).to(torch.bfloat16) if case["tokens"] else g.normal((V, H), 0.02)
    cap = case["capacity"]
    pos = g.ints(case["kv_lo"], case["kv_hi"], B)
    inp = dict(w=w, pos=pos)
    if case["page"]:
        page, per = case["page"], -(-cap // case["page"])
        n_pages = per * B + 3
        inp["kc"], inp["vc"] = (g.normal((L, n_pages, nkv, page, HD)) for _ in range(2))
        inp["table"] = torch.randperm(n_pages, generator=g.g, device="cuda")[:per * B].to(torch.int32).view(B, per).contiguous()
    else:
        inp["kc"], inp["vc"] = (g.normal((L, case["max_batch"], nkv, cap, HD)) for _ in range(2))
    if case["entry"] == "layers":
        inp["x"] = g.normal((B, H)).float()
    elif case["ids"]:
        inp["ids"] = g.ints(0, V - 1, B)
    else:
        inp["x"] = g.normal((B, H))
    return inp


def prepare(case, seed):
    m, B = MODELS[case["model"]], case["batch"]
    s = _inputs(case, seed)
    shape = dict(n_layers=case["layers"], hidden=m["hidden"], n_q_heads=m["nq"], n_kv_heads=m["nkv"], head_dim=HD, ffn=m["ffn"],
                 vocab=case["vocab"], max_batch=case["max_batch"], max_seq=case["capacity"], rms_eps=EPS, rope_theta=THETA)
    s["case"] = case
    s["fleet"] = _Handle(F.fleet_create(shape, s["w"]))
    s["hidden"] = torch.zeros((B, m["hidden"]), device="cuda", dtype=torch.float32)
    s["logits"] = torch.zeros((B, case["vocab"]), device="cuda", dtype=torch.float32) if case["vocab"] else None
    if case["tokens"]:
        s["tok"], s["cur"] = s["ids"].clone(), s["pos"].clone()
        s["out"] = torch.zeros((case["tokens"], B), device="cuda", dtype=torch.int32)
    s["stream"] = torch.cuda.current_stream().cuda_stream
    return s


class _Handle:
    """The library's handle; freed with the state."""

    def __init__(self, f):
        self.f = f
        weakref.finalize(self, F.fleet_destroy, f)


def run(s):
    c, f, B = s["case"], s["fleet"].f, s["case"]["batch"]
    kc, vc, pos, hidden, logits, stream = s["kc"], s["vc"], s["pos"], s["hidden"], s["logits"], s["stream"]
    x, ids = s.get("x"), s.get("ids")
    if c["entry"] == "step":
        F.fleet_decode_step(f, B, x, ids, kc, vc, pos, hidden, logits, stream)
    elif c["entry"] == "static":
        F.fleet_decode_step_static(f, B, x, ids, kc, vc, pos, hidden, logits, stream)
    elif c["entry"] == "layers":
        F.fleet_decode_layers(f, B, 0, c["layers"], x, kc, vc, pos, hidden, logits, stream)
    elif c["entry"] == "paged":
        F.fleet_decode_step_paged(f, B, x, ids, kc, vc, s["table"], c["page"], kc.shape[1], s["table"].shape[1], pos, hidden, logits, stream)
    else:   # the requests' first tokens and lengths, then the call that advances both
        s["tok"].copy_(ids)
        s["cur"].copy_(pos)
        F.fleet_decode_tokens(f, B, s["tok"], kc, vc, s["cur"], c["tokens"], s["out"], hidden, logits, stream)
        return dict(hidden=hidden, logits=logits, k_cache=kc, v_cache=vc, generated=s["out"], tokens=s["tok"], positions=s["cur"])
    out = dict(hidden=hidden, k_cache=kc, v_cache=vc)
    if logits is not None:
        out["logits"] = logits
    return out


def work(case):
    """Every weight read once per step (the steps of one call follow each other), the valid cache
    slots of every sequence read once, the new slot written, inputs and outputs once."""
    m, L, B, V = MODELS[case["model"]], case["layers"], case["batch"], case["vocab"]
    H, nq, nkv, ffn = m["hidden"], m["nq"], m["nkv"], m["ffn"]
    params = L * ((nq + 2 * nkv) * HD * H + nq * HD * H + 3 * ffn * H) + V * H
    steps = max(1, case["tokens"])
    kv = 0.5 * (case["kv_lo"] + case["kv_hi"]) + 0.5 * (steps - 1)
    cache = L * B * 2 * nkv * HD * 2 * (kv + 1)
    io = B * H * 2 + B * H * 4 + B * V * 4
    flops = 2 * params * B + L * B * 4 * nq * HD * (kv + 1)
    return {"bytes": steps * (params * 2 + cache + io), "flops": steps * flops}


def tolerance(case):
    """Two correct implementations round the same operands to bf16 (norm outputs, q, k, v, attention
    output, SwiGLU product) from sums of another order, and differ by flips of these roundings.
    Measured against float64 without any rounding: 0.0008 to 0.006 for one to four layers, 0.018 for
    36 (every flip travels through the layers that follow)."""
    if case["layers"] <= 4:
        return {"rel": 1e-2, "max": 8e-2}
    return {"rel": 5e-2, "max": 3e-1}


def exact(case, seed):
    """The step in float64, without any intermediate rounding; the cache's new slots likewise."""
    s = _inputs(case, seed)
    m, L, B = MODELS[case["model"]], case["layers"], case["batch"]
    H, nq, nkv, ffn = m["hidden"], m["nq"], m["nkv"], m["ffn"]
    grp = nq // nkv
    w, pos = s["w"], s["pos"].long()
    D = torch.float64
    big = s["kc"].numel() > 1 << 28
    kc, vc = (s["kc"], s["vc"]) if big else (s["kc"].double(), s["vc"].double())
    inv = THETA ** (-torch.arange(HD // 2, device="cuda", dtype=D) * 2 / HD)
    rows = torch.arange(B, device="cuda")

    def norm(x, gain):
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * gain.to(D)

    def mul(x, mat):
        return torch.cat([x @ part.to(D).t() for part in mat.split(32768)], 1)

    def rope(x, p):
        a = (p.to(D)[:, None] * inv[None, :])[:, None, :]
        lo, hi = x[..., :HD // 2], x[..., HD // 2:]
        return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)

    def past(c, l, b, n):
        if not case["page"]:
            return c[l, b, :, :n].to(D)
        return c[l, s["table"][b, :-(-n // case["page"])].long()].transpose(0, 1).reshape(nkv, -1, HD)[:, :n].to(D)

    def step(x, p, new_k, new_v):
        for l in range(L):
            qkv = mul(norm(x, w["ln1"][l]), w["wqkv"][l]).view(B, nq + 2 * nkv, HD)
            q = rope(norm(qkv[:, :nq], w["q_norm"][l]), p)
            k = rope(norm(qkv[:, nq:nq + nkv], w["k_norm"][l]), p)
            v = qkv[:, nq + nkv:]
            new_k[l].append(k)
            new_v[l].append(v)
            att = torch.empty((B, nq, HD), device="cuda", dtype=D)
            for b, n in enumerate(s["pos"].tolist()):
                K = torch.cat([past(kc, l, b, n)] + [t[b][:, None] for t in new_k[l]], 1)
                V = torch.cat([past(vc, l, b, n)] + [t[b][:, None] for t in new_v[l]], 1)
                sc = torch.softmax(q[b].view(nkv, grp, HD) @ K.transpose(1, 2).contiguous() / math.sqrt(HD), -1)
                att[b] = (sc @ V).view(nq, HD)
            x = x + mul(att.view(B, -1), w["wo"][l])
            gu = mul(norm(x, w["ln2"][l]), w["wgu"][l])
            gate, up = gu[:, :ffn], gu[:, ffn:]
            x = x + mul(gate / (1 + torch.exp(-gate)) * up, w["wdown"][l])
        return x, (mul(norm(x, w["final_norm"]), w["lm_head"]) if case["vocab"] else None)

    new_k, new_v = [[] for _ in range(L)], [[] for _ in range(L)]
    ids, gen, p = s.get("ids"), [], pos
    for _ in range(max(1, case["tokens"])):
        x0 = w["embed"][ids.long()] if ids is not None else s["x"]
        x, lg = step(x0.to(D), p, new_k, new_v)
        p = p + 1
        if case["tokens"]:
            ids = lg.argmax(1).to(torch.int32)
            gen.append(ids)
    out = dict(hidden=x, k_cache=None, v_cache=None)
    if not big:
        for name, c, new in (("k_cache", kc, new_k), ("v_cache", vc, new_v)):
            for l in range(L):
                for i, t in enumerate(new[l]):
                    slot = pos + i
                    if case["page"]:
                        pg = s["table"][rows, slot // case["page"]].long()
                        c[l][pg, :, slot % case["page"]] = t
                    else:
                        c[l][rows, :, slot] = t
            out[name] = c
    if lg is not None:
        out["logits"] = lg
    if case["tokens"]:
        out.update(generated=torch.stack(gen), tokens=ids, positions=p.to(torch.int32))
    return out
