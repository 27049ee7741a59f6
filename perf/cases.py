"""Performance cases of the serving hot path: what is timed, on which inputs, and what the results should be.

The path is one decoder layer called phase by phase (prefill, a chunk of a prefill over a cached prefix, decode, and
both fused in a mixed step) over a paged KV cache, and the layer stack with embedding and LM head around it. Every case
calls the public entry points as a serving loop does: weights tiled once, a KV pool that outlives the call, a workspace
sized once, one call per layer and step. Lengths are committed once per model step, after every layer, so a call of one
layer leaves them as they were and can be repeated.

Layer shapes are the 8B-shaped, 70B-shaped and tiny fp32 layers of the benchmark and the tests. Prompt and context
lengths follow their laws; batch sizes run from one chat user to the largest batch of the phase sweep (256).

Inputs come from the seed alone: weights N(0, 0.02^2), norm gains 1 + N(0, 0.02^2), activations and cached keys and
values N(0, 1). A pool's pages are handed out in turn to sequences that grow side by side, so that a sequence's pages
lie scattered over the pool, as they do after some time of serving.
"""
import math
import random

import torch

from paper_2608_21719_amd import binding as B

PAGE = 16

#        hidden, q heads, kv heads, head dim, ffn, eps, theta, dtype
SHAPES = {
    "8b": (4096, 32, 8, 128, 14336, 1e-5, 500000.0, "bf16"),
    "70b": (8192, 64, 8, 128, 28672, 1e-5, 500000.0, "bf16"),
    "tiny": (256, 4, 2, 64, 1024, 1e-5, 10000.0, "f32"),
}


class Shape:
    def __init__(self, name):
        (self.hidden, self.n_q, self.n_kv, self.head_dim, self.ffn, self.eps, self.theta, self.dtype) = SHAPES[name]
        self.d_q, self.d_kv = self.n_q * self.head_dim, self.n_kv * self.head_dim
        self.torch_dtype = torch.bfloat16 if self.dtype == "bf16" else torch.float32
        self.elt = 2 if self.dtype == "bf16" else 4

    @property
    def params(self):
        return self.hidden * (self.d_q + 2 * self.d_kv) + self.d_q * self.hidden + 3 * self.hidden * self.ffn


def case(name, shape, **kw):
    c = {"name": name, "shape": shape,
         # new_seqs prompts or chunks of new_lo..new_hi rows behind past_lo..past_hi cached tokens
         "new_seqs": 0, "new_lo": 0, "new_hi": 0, "past_lo": 0, "past_hi": 0,
         # dec_seqs decoding sequences; contexts uniform in ctx_lo..ctx_hi, or log-normal around ctx_median
         # (sigma 0.5) clipped to that range where ctx_median > 0
         "dec_seqs": 0, "ctx_lo": 0, "ctx_hi": 0, "ctx_median": 0,
         "layers": 1, "vocab": 0,  # vocab > 0: the stack of layers with embedding and LM head
         "steps": 0,               # > 0: prefill, then so many decode steps, in one pass
         "len_seed": 1}
    c.update(kw)
    return c


def listed():
    return [
        # one chat user, answer phase: the latency of the smallest step a serving loop makes
        case("decode_8b_b1", "8b", dec_seqs=1, ctx_lo=2048, ctx_hi=2048),
        # the benchmark's answer-phase batch
        case("decode_8b_b64", "8b", dec_seqs=64, ctx_lo=1024, ctx_hi=4096),
        # the largest batch of the phase sweep, contexts of short chats
        case("decode_8b_b256", "8b", dec_seqs=256, ctx_lo=512, ctx_hi=2048),
        # the benchmark's reasoning batch: long log-normal contexts
        case("think_8b_b32", "8b", dec_seqs=32, ctx_lo=4096, ctx_hi=32768, ctx_median=12288),
        # the large layer's decode batch at a fixed context
        case("decode_70b_b64", "70b", dec_seqs=64, ctx_lo=4096, ctx_hi=4096),
        # the benchmark's headline: eight long prompts at once
        case("prefill_8b_8x2048", "8b", new_seqs=8, new_lo=2048, new_hi=2048),
        # one user's question: a single short prompt of an odd length, time to first token
        case("prefill_8b_1x389", "8b", new_seqs=1, new_lo=389, new_hi=389),
        # a few follow-up turns over long cached conversations (chunked prefill)
        case("chunk_8b_3x512_past", "8b", new_seqs=3, new_lo=300, new_hi=512, past_lo=6000, past_hi=12000),
        # the large layer's prefill batch
        case("prefill_70b_8x1024", "70b", new_seqs=8, new_lo=1024, new_hi=1024),
        # new requests join a running reasoning batch
        case("mixed_8b_4x512_b32", "8b", new_seqs=4, new_lo=512, new_hi=512, dec_seqs=32, ctx_lo=4096, ctx_hi=32768,
             ctx_median=12288),
        # the fp32 configuration: prefill, then sixteen decode steps
        case("tiny_f32_4x128_16steps", "tiny", new_seqs=4, new_lo=128, new_hi=128, steps=16),
        # a whole decode step of a small stack with the full vocabulary: embedding, layers, head, greedy token
        case("model_8b_4layers_b8", "8b", dec_seqs=8, ctx_lo=256, ctx_hi=2048, layers=4, vocab=128256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "think", "prefill", "prefill", "chunk", "mixed", "tiny", "model"])
    kw = {"len_seed": rng.randrange(1, 1 << 30)}
    shape = rng.choice(["8b", "8b", "70b"])
    if kind == "decode":
        kw["dec_seqs"] = _log_int(rng, 1, 256)
        kw["ctx_lo"] = _log_int(rng, 16, 2048)
        kw["ctx_hi"] = kw["ctx_lo"] + _log_int(rng, 1, 2048)
    elif kind == "think":
        shape = "8b"
        kw.update(dec_seqs=_log_int(rng, 2, 32), ctx_lo=4096, ctx_hi=32768, ctx_median=_log_int(rng, 6000, 12288))
    elif kind in ("prefill", "chunk"):
        rows = _log_int(rng, 33, 16384 if shape == "8b" else 8192)
        if kind == "chunk":
            rows = min(rows, 4096)
            kw["past_lo"] = _log_int(rng, 16, 8000)
            kw["past_hi"] = kw["past_lo"] + _log_int(rng, 1, 4000)
        kw["new_seqs"] = rng.randint(1, max(1, min(8, rows // 32)))
        kw["new_hi"] = rows // kw["new_seqs"]
        kw["new_lo"] = max(1, int(kw["new_hi"] * rng.uniform(0.3, 1.0)))
    elif kind == "mixed":
        rows = _log_int(rng, 65, 4096 if shape == "8b" else 2048)
        kw["new_seqs"] = rng.randint(1, max(1, min(6, rows // 32)))
        kw["new_hi"] = rows // kw["new_seqs"]
        kw["new_lo"] = max(1, int(kw["new_hi"] * rng.uniform(0.3, 1.0)))
        kw["dec_seqs"] = _log_int(rng, 1, 64)
        kw["ctx_lo"] = _log_int(rng, 64, 6000)
        kw["ctx_hi"] = kw["ctx_lo"] + _log_int(rng, 1, 4000)
    elif kind == "tiny":
        shape = "tiny"
        kw["new_seqs"] = rng.randint(1, 8)
        kw["new_hi"] = _log_int(rng, 5, 256)
        kw["new_lo"] = max(1, int(kw["new_hi"] * rng.uniform(0.3, 1.0)))
        kw["steps"] = rng.randint(1, 16)
    else:
        shape = "8b"
        kw.update(layers=rng.randint(2, 4), vocab=128256)
        if rng.random() < 0.5:
            kw["dec_seqs"] = _log_int(rng, 1, 64)
            kw["ctx_lo"] = _log_int(rng, 16, 1024)
            kw["ctx_hi"] = kw["ctx_lo"] + _log_int(rng, 1, 1024)
        else:
            kw["new_seqs"] = rng.randint(1, 4)
            kw["new_hi"] = _log_int(rng, 33, 700)
            kw["new_lo"] = max(1, int(kw["new_hi"] * rng.uniform(0.3, 1.0)))
    c = case("", shape, **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------- lengths and pages
class Lengths:
    """Cached tokens and new rows of each sequence (chunk sequences first), and the sequence each pool page goes to."""

    def __init__(self, c):
        r = random.Random(c["len_seed"])
        self.n_chunk, self.n_dec = c["new_seqs"], c["dec_seqs"]
        self.past = [r.randint(c["past_lo"], c["past_hi"]) for _ in range(self.n_chunk)]
        self.new = [r.randint(c["new_lo"], c["new_hi"]) for _ in range(self.n_chunk)]
        for _ in range(self.n_dec):
            if c["ctx_median"]:
                x = math.exp(math.log(c["ctx_median"]) + 0.5 * r.gauss(0.0, 1.0))
                x = min(max(int(round(x)), c["ctx_lo"]), c["ctx_hi"])
            else:
                x = r.randint(c["ctx_lo"], c["ctx_hi"])
            self.past.append(x)
            self.new.append(1)
        self.rows = sum(self.new)
        self.pages = [(p + n + c["steps"] + PAGE - 1) // PAGE for p, n in zip(self.past, self.new)]
        self.n_pages = sum(self.pages)
        # page i of the pool belongs to sequence owner[i]: sequences grow side by side
        self.owner = [s for s, n in enumerate(self.pages) for _ in range(n)]
        r.shuffle(self.owner)
        self.table = [[] for _ in self.pages]
        for page, s in enumerate(self.owner):
            self.table[s].append(page)


# ---------------------------------------------------------------- inputs from the seed
class Inputs:
    """Row-major weights, activations (or token ids) and the pool's contents, on the GPU."""

    def __init__(self, c, seed):
        s = Shape(c["shape"])
        L = Lengths(c)
        g = torch.Generator(device="cuda").manual_seed(seed)

        def normal(*shape, std=1.0, mean=0.0):
            t = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
            if std != 1.0:
                t.mul_(std)
            if mean:
                t.add_(mean)
            return t.to(s.torch_dtype)

        self.weights = []
        for _ in range(c["layers"]):
            self.weights.append({
                "attn_norm": normal(s.hidden, std=0.02, mean=1.0),
                "qkv": normal(s.d_q + 2 * s.d_kv, s.hidden, std=0.02),
                "o": normal(s.hidden, s.d_q, std=0.02),
                "ffn_norm": normal(s.hidden, std=0.02, mean=1.0),
                "gate": normal(s.ffn, s.hidden, std=0.02),
                "up": normal(s.ffn, s.hidden, std=0.02),
                "down": normal(s.hidden, s.ffn, std=0.02),
            })
        # [layers, pages, kv heads, K block | V^T block]; prompts start from an empty cache
        shape = (c["layers"], L.n_pages, s.n_kv, 2, PAGE * s.head_dim)
        if any(L.past):
            self.pool = normal(*shape)
        else:
            self.pool = torch.zeros(shape, dtype=s.torch_dtype, device="cuda")
        if c["vocab"]:
            self.embed = normal(c["vocab"], s.hidden, std=0.02)
            self.head = normal(c["vocab"], s.hidden, std=0.02)
            self.final_norm = normal(s.hidden, std=0.02, mean=1.0)
            self.tokens = torch.randint(0, c["vocab"], (L.rows,), generator=g, device="cuda", dtype=torch.int32)
        else:
            self.x = normal(L.rows, s.hidden)
            self.step_x = [normal(len(L.new), s.hidden) for _ in range(c["steps"])]
        self.shape, self.lengths = s, L


# ---------------------------------------------------------------- what a serving program holds before the call
class State:
    pass


def prepare(case, seed):
    c, st = case, State()
    i = Inputs(c, seed)
    s, L = i.shape, i.lengths
    code = B.PS_BF16 if s.dtype == "bf16" else B.PS_F32

    def tiled(w):
        n, k = w.shape
        out = torch.empty(B.tiled_weight_elems(n, k), dtype=w.dtype, device="cuda")
        B.op_tile_weight(code, n, k, w, out)
        return out

    st.weights = []
    for k, w in enumerate(i.weights):
        # gate and up rows interleaved in blocks of 32
        gate_up = torch.stack([w["gate"].view(-1, B.GATE_UP_BLOCK, s.hidden), w["up"].view(-1, B.GATE_UP_BLOCK, s.hidden)],
                              dim=1).view(2 * s.ffn, s.hidden)
        t = [w["attn_norm"], tiled(w["qkv"]), tiled(w["o"]), w["ffn_norm"], tiled(gate_up), tiled(w["down"])]
        st.weights.append((t, B.layer_weights(*t)))
        i.weights[k] = None
    st.cfg = B.make_cfg(_CfgShape(s))
    st.pool = i.pool
    n, max_pages = len(L.new), max(L.pages)
    st.kv = B.KV(st.cfg, c["layers"], L.n_pages, n, max_pages, st.pool, seed=0)
    seqs = [st.kv.open() for _ in range(n)]
    have = [0] * n
    for q in L.owner:
        have[q] += 1
        st.kv.alloc(seqs[q], have[q] * PAGE)
    st.kv.commit(seqs, L.past)
    st.chunk, st.chunk_tok, st.dec = seqs[:L.n_chunk], L.new[:L.n_chunk], seqs[L.n_chunk:]
    st.case, st.seqs = c, seqs
    if c["vocab"]:
        st.embed, st.head, st.final_norm, st.tokens = i.embed, tiled(i.head), i.final_norm, i.tokens
        st.model = B.Model(st.cfg, [w for _, w in st.weights], c["vocab"], st.embed, st.final_norm, st.head)
        nbytes = B.Model.workspace_bytes(st.cfg, c["vocab"], L.rows, n, max_pages)
        st.next = torch.empty(n, dtype=torch.int32, device="cuda")
        st.logits = torch.empty((n, c["vocab"]), dtype=torch.float32, device="cuda")
    else:
        st.layer = B.Layer(st.cfg)
        nbytes = B.Layer.workspace_bytes(st.cfg, L.rows, n, max_pages)
        st.x, st.out = i.x, torch.empty_like(i.x)
        st.step_x, st.step_out = i.step_x, [torch.empty_like(x) for x in i.step_x]
    st.ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    return st


class _CfgShape:
    """The attributes binding.make_cfg reads."""

    def __init__(self, s):
        self.hidden, self.n_q, self.n_kv, self.head_dim, self.ffn = s.hidden, s.n_q, s.n_kv, s.head_dim, s.ffn
        self.eps, self.theta, self.dtype = s.eps, s.theta, s.dtype


def run(state):
    st = state
    if st.case["vocab"]:
        # the greedy tokens are the logits' argmax; a near tie would turn one on any change of rounding, so the
        # logits stand for them
        if st.chunk:
            st.model.prefill(st.kv, st.chunk, st.chunk_tok, st.tokens, st.next, st.ws, st.logits)
        else:
            st.model.decode_step(st.kv, B.PS_PHASE_ANSWER, st.dec, st.tokens, st.next, st.ws, st.logits)
        return {"logits": st.logits, "kv": st.pool}
    w = st.weights[0][1]
    if st.case["steps"]:
        st.layer.prefill(w, st.kv, 0, st.chunk, st.chunk_tok, st.x, st.out, st.ws)
        st.kv.commit(st.chunk, st.chunk_tok)
        for x, out in zip(st.step_x, st.step_out):
            st.layer.decode_step(w, st.kv, 0, B.PS_PHASE_THINK, st.chunk, x, out, st.ws)
            st.kv.commit(st.chunk, [1] * len(st.chunk))
        for q in st.chunk:
            st.kv.truncate(q, 0)
        return {"x": st.out, "steps": st.step_out, "kv": st.pool}
    if st.chunk and st.dec:
        st.layer.mixed_step(w, st.kv, 0, st.chunk, st.chunk_tok, st.dec, st.x, st.out, st.ws)
    elif st.chunk:
        st.layer.prefill(w, st.kv, 0, st.chunk, st.chunk_tok, st.x, st.out, st.ws)
    else:
        phase = B.PS_PHASE_THINK if st.case["ctx_median"] else B.PS_PHASE_ANSWER
        st.layer.decode_step(w, st.kv, 0, phase, st.dec, st.x, st.out, st.ws)
    return {"x": st.out, "kv": st.pool}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    c, s, L = case, Shape(case["shape"]), Lengths(case)
    n = len(L.new)
    rows = L.rows + c["steps"] * n
    pairs = sum(p * t + t * (t + 1) // 2 for p, t in zip(L.past, L.new))
    past = list(L.past)
    kv_read = sum(L.past)  # cached tokens each attention reads once
    if c["steps"]:
        past = [p + t for p, t in zip(L.past, L.new)]
        for _ in range(c["steps"]):
            pairs += sum(p + 1 for p in past)
            kv_read += sum(past)
            past = [p + 1 for p in past]
    passes = 1 + c["steps"]
    nbytes = c["layers"] * (passes * s.params * s.elt + (kv_read + rows) * 2 * s.d_kv * s.elt) + 2 * rows * s.hidden * s.elt
    flops = c["layers"] * (2 * rows * s.params + 4 * s.d_q * pairs)
    if c["vocab"]:
        nbytes += c["vocab"] * s.hidden * s.elt + n * c["vocab"] * 4 - rows * s.hidden * s.elt
        flops += 2 * n * c["vocab"] * s.hidden
    return {"bytes": nbytes, "flops": flops}


# Against 64 bits the fp32 layer is 3e-7 off, a bf16 layer 3.2e-3 to 4.8e-3 (8B shape) and 1.1e-2 (70B shape, whose wider
# FFN carries the rounding of its product into the output), the stack's logits 1.2e-2 to 1.6e-2. Another order of the sums
# turns bf16 roundings on the way, so two correct runs differ by up to as much; the 8B layer and the fp32 layer get a
# margin over that. Elements go as far as six times the root mean square, and a large one by its own last bit.
def tolerance(case):
    if case["shape"] == "tiny":
        return {"rel": 2e-6, "max": 1e-4}
    if case["vocab"]:
        return {"rel": 3e-2, "max": 0.4}
    return {"rel": 2e-2, "max": 0.2} if case["shape"] == "70b" else {"rel": 1e-2, "max": 0.1}


# ---------------------------------------------------------------- the same in 64 bits
def _rmsnorm(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _linear(x, w):
    return x @ w.double().T


def _rope(x, pos, theta):
    """Rotate-half pairs (j, j + hd/2), angle pos * theta^(-2j/hd); x [rows, heads, hd]."""
    half = x.shape[-1] // 2
    j = torch.arange(half, dtype=torch.float64, device=x.device)
    a = (pos.double()[:, None] * theta ** (-2.0 * j / (2 * half)))[:, None, :]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], dim=-1)


def _layer64(s, w, pool, table, past, new, x):
    """One layer over the rows of x (grouped by sequence); pool [pages, kv heads, 2, 16 hd] in 64 bits is updated."""
    G, hd, dev = s.n_q // s.n_kv, s.head_dim, x.device
    pos = torch.cat([torch.arange(p, p + t, device=dev) for p, t in zip(past, new)])
    qkv = _linear(_rmsnorm(x, w["attn_norm"], s.eps), w["qkv"])
    q = _rope(qkv[:, :s.d_q].reshape(-1, s.n_q, hd), pos, s.theta)
    k = _rope(qkv[:, s.d_q:s.d_q + s.d_kv].reshape(-1, s.n_kv, hd), pos, s.theta)
    v = qkv[:, s.d_q + s.d_kv:].reshape(-1, s.n_kv, hd)
    page = torch.cat([torch.tensor(table[b], device=dev)[torch.arange(p, p + t, device=dev) // PAGE]
                      for b, (p, t) in enumerate(zip(past, new))])
    pool[:, :, 0].view(-1, s.n_kv, PAGE, hd).transpose(1, 2)[page, pos % PAGE] = k
    pool[:, :, 1].view(-1, s.n_kv, hd, PAGE).permute(0, 3, 1, 2)[page, pos % PAGE] = v
    o = torch.empty_like(q)
    r0 = 0
    for b, (p, t) in enumerate(zip(past, new)):
        n = p + t
        blk = pool[torch.tensor(table[b][:(n + PAGE - 1) // PAGE], device=dev)]
        kk = blk[:, :, 0].reshape(-1, s.n_kv, PAGE, hd).permute(1, 0, 2, 3).reshape(s.n_kv, -1, hd)[:, :n].contiguous()
        vv = blk[:, :, 1].reshape(-1, s.n_kv, hd, PAGE).permute(1, 0, 3, 2).reshape(s.n_kv, -1, hd)[:, :n].contiguous()
        qq = q[r0:r0 + t].reshape(t, s.n_kv, G, hd).permute(1, 2, 0, 3).reshape(s.n_kv, G * t, hd)
        sc = torch.bmm(qq, kk.transpose(1, 2).contiguous()) / math.sqrt(hd)
        if t > 1:
            hidden = torch.arange(n, device=dev)[None, :] > torch.arange(p, n, device=dev)[:, None]
            sc.view(s.n_kv, G, t, n).masked_fill_(hidden, -math.inf)
        out = torch.bmm(torch.softmax(sc, dim=-1), vv)
        o[r0:r0 + t] = out.view(s.n_kv, G, t, hd).permute(2, 0, 1, 3).reshape(t, s.n_q, hd)
        r0 += t
    h = x + _linear(o.reshape(-1, s.d_q), w["o"])
    hn = _rmsnorm(h, w["ffn_norm"], s.eps)
    m = torch.nn.functional.silu(_linear(hn, w["gate"])) * _linear(hn, w["up"])
    return h + _linear(m, w["down"])


def exact(case, seed):
    c = case
    i = Inputs(c, seed)
    s, L = i.shape, i.lengths
    pool = i.pool.double()
    if c["vocab"]:
        x = i.embed[i.tokens.long()].double()
        for k, w in enumerate(i.weights):
            x = _layer64(s, w, pool[k], L.table, L.past, L.new, x)
        last = torch.tensor(L.new, device=x.device).cumsum(0) - 1
        return {"logits": _linear(_rmsnorm(x[last], i.final_norm, s.eps), i.head), "kv": pool}
    x = _layer64(s, i.weights[0], pool[0], L.table, L.past, L.new, i.x.double())
    if not c["steps"]:
        return {"x": x, "kv": pool}
    steps, past = [], [p + t for p, t in zip(L.past, L.new)]
    for sx in i.step_x:
        steps.append(_layer64(s, i.weights[0], pool[0], L.table, past, [1] * len(past), sx.double()))
        past = [p + 1 for p in past]
    return {"x": x, "steps": steps, "kv": pool}
