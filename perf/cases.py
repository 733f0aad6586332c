"""Performance cases: the calls an edit-oriented speculative decoder makes.

A case is one call of the verification library on a model that is already
loaded, over a committed KV cache: a prompt prefill, one greedy step, a linear
or tree draft verified in one block, a batch of sequences, entropy-aware
(top-k) and stochastic verification.  Models are the shapes of
``workloads.configs`` with random weights; the 7B and 33B ones keep their full
width and vocabulary and run a few layers (every layer is the same work, and
a layer's share of a call is what the whole model repeats), the 1B model and
the small fp32 one run whole.

``prepare`` builds the engine, installs a random committed cache (or the
prompt) and runs the call once, as a serving loop that has been running does;
``run`` rewinds the sequences to that cache and makes the call again.  Outputs
are the call's results, the logits of the block and the whole KV pool.  The
last two stay where the engine keeps them on the GPU: the pool and the
workspace are the caller's own buffers, and ``prepare`` finds the logits in
the workspace by comparing it with what ``Engine.logits`` returns.
"""

from __future__ import annotations

import math
from collections import OrderedDict

import numpy as np
import torch

import paper_2506_02780_amd as ee
from workloads import get_shape, random_tree, zipf_tokens

PAGE = 64            # KV positions per page
WEIGHT_SEED = 1234   # the model is the same in every call; prompts, caches and drafts are not
STD = 0.02

# Layers run per model (the small and the 1B model are whole).
LAYERS = {"tiny": 2, "1b": 16, "7b": 4, "33b": 1}


# ------------------------------------------------------------------- cases --

def _case(name=None, *, model, call, ctx, k=0, seqs=1, k_max=64, top_k=0, temperature=0.0):
    c = {"model": model, "call": call, "ctx": ctx, "k": k, "seqs": seqs, "k_max": k_max, "top_k": top_k,
         "temperature": temperature}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: 9 rows of a two-layer fp32 model, where launches and latency are all
        _case("tiny fp32 verify k8", model="tiny", call="verify", ctx=64, k=8),
        # plain greedy decoding at an edit position: one row, every weight read for it
        _case("7b greedy step", model="7b", call="verify", ctx=2048, k=0),
        # the Reuse step: 32 tokens of the original code verified in one block
        _case("7b reuse k32", model="7b", call="verify", ctx=2048, k=32),
        # the longest Reuse draft an engine takes by default, at an odd context
        _case("7b reuse k64", model="7b", call="verify", ctx=1999, k=64),
        # a draft tree of 64 nodes (depth 8, branching 3) verified in one pass
        _case("7b tree 64", model="7b", call="tree", ctx=2048, k=64),
        # a long span of the original code in one block
        _case("7b reuse k512", model="7b", call="verify", ctx=2048, k=512, k_max=512),
        # the prompt of an edit task, in blocks of the longest draft
        _case("7b prefill 2048", model="7b", call="prefill", ctx=2048, k_max=512),
        # a prompt on an engine with the default block size, whole 1B model
        _case("1b prefill 1000", model="1b", call="prefill", ctx=1000, k_max=64),
        # a whole small model: sixteen layers of few bytes each
        _case("1b reuse k16", model="1b", call="verify", ctx=1024, k=16),
        # four edit sequences at once on the widest model
        _case("33b batch 4 x k64", model="33b", call="verify", ctx=4096, k=64, seqs=4),
        # Generate steps of twelve sequences: 7 tokens of a draft model each, entropy-aware acceptance
        _case("7b top5 12 x k7", model="7b", call="topk", ctx=500, k=7, seqs=12, top_k=5),
        # stochastic verification late in a long context
        _case("7b sample k24", model="7b", call="sample", ctx=7900, k=24, temperature=0.8),
    ]


def draw(rng):
    def spread(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(["step", "verify", "verify", "tree", "long", "prefill", "batch", "topk", "sample"])
    model = rng.choice(["tiny", "1b", "7b", "7b"])
    ctx = spread(16, 7900 if model == "7b" else 4000)
    if kind == "step":
        return _case(model=model, call="verify", ctx=ctx, k=0)
    if kind == "verify":
        return _case(model=model, call="verify", ctx=ctx, k=rng.randint(1, 64))
    if kind == "tree":
        return _case(model=model, call="tree", ctx=ctx, k=rng.randint(8, 64))
    if kind == "long":
        return _case(model=model, call="verify", ctx=min(ctx, 2048), k=spread(65, 500), k_max=512)
    if kind == "prefill":
        return _case(model=model, call="prefill", ctx=spread(8, 2000), k_max=rng.choice([32, 64, 512]))
    if kind == "batch":
        if rng.random() < 0.4:
            return _case(model="33b", call="verify", ctx=spread(16, 3000), k=rng.randint(0, 60),
                         seqs=rng.randint(2, 4))
        return _case(model=model, call="verify", ctx=spread(16, 1500), k=rng.randint(0, 32), seqs=rng.randint(2, 12))
    if kind == "topk":
        return _case(model=model, call="topk", ctx=spread(16, 1500), k=rng.randint(1, 32), seqs=rng.randint(1, 8),
                     top_k=rng.randint(2, 8))
    return _case(model=model, call="sample", ctx=ctx, k=rng.randint(0, 32), temperature=rng.choice([0.3, 0.8, 1.0]))


# ------------------------------------------------------------------ models --

def _shape(model):
    return get_shape(model, n_layers=LAYERS[model])


class _Weights:
    """Random weights of one model, drawn on the GPU from a fixed seed and held
    on the host in the layout ``Engine`` takes."""

    def __init__(self, s):
        g = torch.Generator(device="cuda")
        g.manual_seed(WEIGHT_SEED)
        dt = torch.bfloat16 if s.dtype == "bf16" else torch.float32

        def mat(rows, cols):
            t = torch.empty(rows, cols, device="cuda", dtype=torch.float32).normal_(0.0, STD, generator=g).to(dt)
            return t.view(torch.int16).cpu().numpy().view(np.uint16) if s.dtype == "bf16" else t.cpu().numpy()

        def gain():
            return (1.0 + 0.1 * torch.randn(s.d_model, device="cuda", generator=g)).cpu().numpy()

        d, qd, kd, f = s.d_model, s.q_dim, s.kv_dim, s.ffn
        self.embed, self.lm_head, self.final_gain = mat(s.vocab, d), mat(s.vocab, d), gain()
        self._layers = [dict(wq=mat(qd, d), wk=mat(kd, d), wv=mat(kd, d), wo=mat(d, qd), w_gate=mat(f, d),
                             w_up=mat(f, d), w_down=mat(d, f), attn_gain=gain(), ffn_gain=gain())
                        for _ in range(s.n_layers)]

    def layer(self, l):
        return self._layers[l]


_loaded: "OrderedDict[str, _Weights]" = OrderedDict()


def _weights(model):
    """The host copy of a model's weights (the last three models are kept)."""
    if model not in _loaded:
        _loaded[model] = _Weights(_shape(model))
        while len(_loaded) > 3:
            _loaded.popitem(last=False)
    _loaded.move_to_end(model)
    return _loaded[model]


# ------------------------------------------------------------------ inputs --

def _max_ctx(case):
    return min(8192, case["ctx"] + case["k"] + 66)


def _inputs(case, seed):
    """Everything a call takes, from the seed alone."""
    s = _shape(case["model"])
    x = {"tokens": [zipf_tokens(s.vocab, case["ctx"] if case["call"] == "prefill" else case["k"] + 1,
                                seed=1000 * seed + b) for b in range(case["seqs"])]}
    if case["call"] == "tree":
        depth = 8 if case["k"] >= 32 else 4
        x["parent"] = random_tree(case["k"], max_depth=depth, max_branch=3, seed=seed, require_full_depth=False)
    if case["call"] == "sample":
        r = np.random.Generator(np.random.PCG64(seed))
        x["eps"], x["u"] = r.random(case["k"], dtype=np.float32), r.random(case["k"] + 1, dtype=np.float32)
        x["eps"], x["u"] = np.minimum(x["eps"], np.float32(0.999999)), np.minimum(x["u"], np.float32(0.999999))
    return x


def _cache(case, seed, b):
    """Committed keys and values of sequence b, [layers, ctx, kv heads, head dim] on the GPU."""
    s = _shape(case["model"])
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * seed + b)
    dt = torch.bfloat16 if s.dtype == "bf16" else torch.float32
    dims = (s.n_layers, case["ctx"], s.n_kv_heads, s.head_dim)
    return [torch.randn(dims, device="cuda", generator=g).to(dt) for _ in range(2)]


def _host_bits(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.cpu().numpy()


class _State:
    def __init__(self, case, seed):
        s = _shape(case["model"])
        self.case, self.x = case, _inputs(case, seed)
        self.eng = ee.Engine(s, _weights(case["model"]), max_ctx=_max_ctx(case), max_seqs=case["seqs"],
                             k_max=case["k_max"])
        if case["call"] != "prefill":
            for b in range(case["seqs"]):
                k, v = _cache(case, seed, b)
                self.eng.load_kv(b, _host_bits(k), _host_bits(v), int(self.x["tokens"][b][0]))
        self.kv = self.eng.kv_pool.view(torch.bfloat16 if s.dtype == "bf16" else torch.float32)
        self.call()
        self.logits = self._find_logits()

    def _find_logits(self):
        """The block's logits in the engine's workspace."""
        want = torch.from_numpy(self.eng.logits()).to(self.eng.device)
        ws = self.eng.workspace.view(torch.float32)
        head = want[0, :4]
        hits = (ws[:-4] == head[0]).nonzero().flatten()
        hits = hits[(ws[hits[:, None] + torch.arange(4, device=ws.device)] == head).all(1)]
        for h in hits.tolist():
            view = ws[h:h + want.numel()]
            if view.numel() == want.numel() and torch.equal(view.view_as(want), want):
                return view.view_as(want)
        raise RuntimeError("the block's logits are not in the workspace")

    def call(self):
        c, x, eng = self.case, self.x, self.eng
        if c["call"] == "prefill":
            if eng.seq_state(0)[0]:
                eng.rollback(0, 0, -1)
            return {"next": eng.prefill(0, x["tokens"][0])}
        for b in reversed(range(c["seqs"])):
            eng.rollback(b, c["ctx"], int(x["tokens"][b][0]))
        drafts = [t[1:] for t in x["tokens"]]
        if c["call"] == "topk":
            res = eng.verify_topk(list(range(c["seqs"])), drafts, c["top_k"])
            return {"accepted": [r[0] for r in res], "next": [r[1] for r in res], "thresholds": [r[2] for r in res]}
        if c["call"] == "sample":
            a, nxt = eng.verify_sample(0, drafts[0], x["eps"], x["u"], temperature=c["temperature"])
            return {"accepted": a, "next": nxt}
        if c["seqs"] > 1:
            res = eng.verify_batch(list(range(c["seqs"])), drafts)
            return {"accepted": [r[0] for r in res], "next": [r[1] for r in res]}
        a, nxt, nodes = eng.verify(0, drafts[0], x.get("parent"))
        return {"accepted": a, "next": nxt}


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    return {**state.call(), "logits": state.logits, "kv": state.kv}


# -------------------------------------------------------------------- work --

def work(case):
    s = _shape(case["model"])
    esz = 2 if s.dtype == "bf16" else 4
    linear = s.n_layers * ((s.q_dim + 2 * s.kv_dim) * s.d_model + s.d_model * s.q_dim + 3 * s.ffn * s.d_model)
    head = s.vocab * s.d_model
    kv_row = 2 * s.kv_dim * esz * s.n_layers
    if case["call"] == "prefill":
        # weights are read once, the cache is written once; only the last row's logits are asked for
        n = case["ctx"]
        seen = n * (n + 1) // 2
        flops = 2 * n * linear + 2 * head + 4 * s.n_layers * s.q_dim * seen
        return {"bytes": esz * (linear + head + n * s.d_model) + n * kv_row + 4 * s.vocab, "flops": flops}
    t, n, b = case["k"] + 1, case["ctx"], case["seqs"]
    rows = b * t
    seen = b * (t * n + t * (t + 1) // 2)
    flops = 2 * rows * (linear + head) + 4 * s.n_layers * s.q_dim * seen
    return {"bytes": esz * (linear + head + rows * s.d_model) + b * (n + t) * kv_row + 4 * rows * s.vocab,
            "flops": flops}


def tolerance(case):
    if _shape(case["model"]).dtype == "f32":
        # measured against exact(): 3e-7 to 4e-7
        return {"rel": 2e-6, "max": 5e-5}
    # measured against exact(), which rounds nothing to bf16: logits 0.009 to 0.016, keys and values up to 0.009; a
    # float32-sized change at any place flips a few bf16 roundings per layer, each of which moves the values after it
    return {"rel": 2e-2, "max": 0.3}


# ------------------------------------------------------------------- exact --

def _f64(a, s):
    t = torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16) if s.dtype == "bf16" else torch.from_numpy(a).cuda()
    return t.double()


def _rms(h, gain, eps):
    return h / torch.sqrt((h * h).mean(-1, keepdim=True) + eps) * gain


def _rotate(x, pos, theta):
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * theta ** (-2.0 * torch.arange(half, device=x.device).double() / x.shape[-1])
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)


def _attend(q, k, v, mask):
    """q [T, H, D], k and v [N, Hkv, D], mask [T, N] (seen keys) -> [T, H * D]."""
    t, h, d = q.shape
    rep = h // k.shape[1]
    out = torch.empty_like(q)
    for g in range(k.shape[1]):
        qg = q[:, g * rep:(g + 1) * rep]
        for j in range(rep):
            sc = (qg[:, j] @ k[:, g].t().contiguous()) / math.sqrt(d)
            out[:, g * rep + j] = torch.softmax(sc.masked_fill(~mask, -math.inf), -1) @ v[:, g]
    return out.reshape(t, h * d)


def exact(case, seed):
    """The same call in float64 with no rounding in between: logits and KV pool."""
    s, w, x = _shape(case["model"]), _weights(case["model"]), _inputs(case, seed)
    dev = torch.device("cuda")
    pages = (_max_ctx(case) + PAGE - 1) // PAGE * case["seqs"]
    pool = torch.zeros(s.n_layers, pages, 2, s.n_kv_heads, PAGE * s.head_dim, dtype=torch.float64, device=dev)
    n = 0 if case["call"] == "prefill" else case["ctx"]
    nt = len(x["tokens"][0])
    # pages in the order the calls take them: the caches, then what each block needs beyond them
    free, page_of = 0, []
    for b in range(case["seqs"]):
        held = (n + PAGE - 1) // PAGE
        page_of.append(list(range(free, free + held)))
        free += held
    for b in range(case["seqs"]):
        more = (n + nt + PAGE - 1) // PAGE - len(page_of[b])
        page_of[b] += range(free, free + more)
        free += more
    block = case["k_max"] + 1 if case["call"] == "prefill" else nt
    first = (nt - 1) // block * block          # the block whose logits are returned
    logits = []
    for b in range(case["seqs"]):
        mask = torch.ones(nt, n + nt, dtype=torch.bool, device=dev)
        pos = n + torch.arange(nt, device=dev)
        if case["call"] == "tree":
            own = torch.zeros(nt, nt, dtype=torch.bool)
            depth = [0] * nt
            own[:, 0] = True
            for i, p in enumerate(x["parent"]):
                own[i + 1] |= own[p + 1]
                own[i + 1, i + 1] = True
                depth[i + 1] = depth[p + 1] + 1
            mask[:, n:] = own.to(dev)
            pos = n + torch.tensor(depth, device=dev)
        else:
            mask[:, n:] = torch.tril(mask[:, n:])
        toks = torch.from_numpy(x["tokens"][b].astype(np.int64)).to(dev)
        h = _f64(w.embed, s)[toks]
        cache = _cache(case, seed, b) if n else None
        new = []
        for l in range(s.n_layers):
            lw = w.layer(l)
            a = _rms(h, _f32(lw["attn_gain"]), s.rms_eps)
            q = (a @ _f64(lw["wq"], s).t()).view(nt, s.n_heads, s.head_dim)
            k = (a @ _f64(lw["wk"], s).t()).view(nt, s.n_kv_heads, s.head_dim)
            v = (a @ _f64(lw["wv"], s).t()).view(nt, s.n_kv_heads, s.head_dim)
            q, k = _rotate(q, pos, s.rope_theta), _rotate(k, pos, s.rope_theta)
            if n:
                k, v = (torch.cat([c[l].double(), y]) for c, y in zip(cache, (k, v)))
            new.append((k, v))
            h = h + _attend(q, k, v, mask) @ _f64(lw["wo"], s).t()
            a = _rms(h, _f32(lw["ffn_gain"]), s.rms_eps)
            z = torch.nn.functional.silu(a @ _f64(lw["w_gate"], s).t()) * (a @ _f64(lw["w_up"], s).t())
            h = h + z @ _f64(lw["w_down"], s).t()
        lg = _rms(h[first:], _f32(w.final_gain), s.rms_eps) @ _f64(w.lm_head, s).t()
        logits.append(lg)
        moved = []                                 # accepted tree rows move to the slots behind the pending row
        if case["call"] == "tree":
            best, cur = lg.argmax(-1).tolist(), 0
            while True:
                hit = [i + 1 for i, p in enumerate(x["parent"]) if p + 1 == cur and int(toks[i + 1]) == best[cur]]
                if not hit:
                    break
                cur = hit[0]
                moved.append(cur)
        pg = torch.tensor(page_of[b], device=dev)
        for l, (k, v) in enumerate(new):
            if moved:
                rows = torch.tensor(moved, device=dev) + n
                k[n + 1:n + 1 + len(moved)], v[n + 1:n + 1 + len(moved)] = k[rows].clone(), v[rows].clone()
            pad = len(page_of[b]) * PAGE - k.shape[0]
            k, v = (torch.nn.functional.pad(y, (0, 0, 0, 0, 0, pad)).view(-1, PAGE, s.n_kv_heads, s.head_dim)
                    for y in (k, v))
            pool[l, pg, 0] = k.permute(0, 2, 1, 3).reshape(len(pg), s.n_kv_heads, -1)
            pool[l, pg, 1] = v.permute(0, 2, 3, 1).reshape(len(pg), s.n_kv_heads, -1)
    return {"logits": torch.cat(logits), "kv": pool.reshape(-1)}


def _f32(a):
    return torch.from_numpy(np.asarray(a)).cuda().double()
