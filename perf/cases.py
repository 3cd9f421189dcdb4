"""The work that programs have this library do, as cases with inputs, one pass, its exact result and its cost.

Every case is a model shape, a number of sequences with their contexts, and one operation through the entry points of
``paper_2609_36590_amd.binding``:

* ``verify``   one verification of k drafts per sequence (k + 1 rows each) with the logits of every row;
* ``draft``    k drafting steps of the decoder layers and the LM head, with the logits of every step;
* ``tree``     one verification of a packed draft tree with the logits of every node;
* ``prefill``  the prompts' prefill and the first verification after it (time to the first tokens), with its logits;
* ``spec``     the forward pass of the drafting objective: logits and negative log-likelihood of every row;
* ``generate`` prefill and draft-verify rounds replayed from a HIP graph, then one drafting step's logits.

Most cases run a few layers of a model's real widths, so that each kernel's share and rounding stay visible; a small
vocabulary leaves the LM head out of a case about the layers. ``verify`` and ``tree`` cases score rows after a
sequence that has reached its token limit: the whole pass runs, and nothing is committed, so a pass can be repeated.

Weights are random with residual projections scaled so that the layers outweigh the embedding in the residual stream
a few to one: the most likely token is then clear of the others (as a trained model's is), and no token that is
fed back hangs on a rounding.
"""
import math
import random

import numpy as np
import torch

from paper_2609_36590_amd import binding

# widths of the repository's model configurations
W4B = dict(hidden=2560, heads=32, kv_heads=8, head_dim=128, ffn=9728, rope_base=1e6, dtype="bf16")
W28L = dict(hidden=2048, heads=16, kv_heads=8, head_dim=128, ffn=6144, rope_base=1e6, dtype="bf16")
WTINY = dict(hidden=256, heads=4, kv_heads=4, head_dim=64, ffn=1024, rope_base=1e4, dtype="f32")
VOCAB, SMALL = 151936, 1024
EPS = 1e-6


def _case(name, op, widths, layers, dec, vocab, lo, hi, batch, k, **more):
    c = dict(op=op, layers=layers, dec=dec, vocab=vocab, lo=lo, hi=hi, batch=batch, k=k, **widths, **more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a toy fp32 model, where launches and host latency are all there is
        _case("verify_tiny_f32", "verify", WTINY, 4, 2, SMALL, 32, 32, 1, 4),
        # one sequence's verification at an ordinary context, the layers' share: latency-critical decoding
        _case("verify_b1", "verify", W4B, 4, 2, SMALL, 1024, 1024, 1, 4),
        # a batch of 8 ragged sequences (40 rows): throughput decoding
        _case("verify_b8", "verify", W4B, 4, 2, SMALL, 256, 2048, 8, 4),
        # long context: attention over 16k positions
        _case("verify_16k", "verify", W4B, 2, 1, SMALL, 16384, 16384, 1, 4),
        # the drafter: two layers and the full LM head, one row at a time
        _case("draft_b1", "draft", W4B, 2, 2, VOCAB, 1024, 1024, 1, 4),
        # drafting for a batch
        _case("draft_b8_28l", "draft", W28L, 2, 2, VOCAB, 100, 900, 8, 2),
        # dynamic drafting's tree verification: 31 nodes, the LM head over all of them
        _case("tree_31", "tree", W28L, 4, 2, VOCAB, 700, 700, 1, 6, nodes=31),
        # a prompt's prefill, the layers' share
        _case("prefill_1k", "prefill", W4B, 4, 2, SMALL, 1024, 1024, 1, 4),
        # a batch of short ragged prompts
        _case("prefill_b4", "prefill", W28L, 4, 2, SMALL, 20, 500, 4, 2),
        # a long document's prefill
        _case("prefill_16k", "prefill", W4B, 2, 1, SMALL, 16384, 16384, 1, 0),
        # the drafting objective over a training sequence: prefill, decoder pass, logits of every row
        _case("spec_1k", "spec", W4B, 2, 1, VOCAB, 1024, 1024, 1, 0, block=4),
        # a whole call on the whole model: prompt in, tokens out
        _case("generate_4b", "generate", W4B, 36, 2, VOCAB, 1024, 1024, 1, 4, new=40),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["verify", "verify", "draft", "tree", "prefill", "prefill", "spec", "generate"])
    w = rng.choice([W4B, W4B, W28L, WTINY])
    tiny = w is WTINY
    layers = rng.randint(2, 4)
    dec = rng.randint(1, layers)
    head = rng.random() < 0.4 and not tiny
    vocab = VOCAB if head else 16 * rng.randint(32, 512)
    batch, k, more = 1, rng.randint(0 if op in ("verify", "prefill", "generate") else 1, 8), {}
    hi = _log_int(rng, 16, 1500 if tiny else 6000)
    if op in ("verify", "draft", "prefill", "generate") and rng.random() < 0.5:
        batch = rng.randint(2, 8)
        k = rng.randint(0 if op in ("verify", "prefill", "generate") else 1, 64 // batch - 1 if batch > 4 else 8)
        hi = min(hi, 2048)
    if op == "tree":
        nodes = rng.randint(2, 64)
        k = rng.randint(1, min(8, nodes - 1))
        more["nodes"] = nodes
    if op == "spec":
        more["block"] = rng.randint(1, 16)
        k = 0
        hi = min(hi, 1024 if head else 2048)
    if op == "generate":
        more["new"] = rng.randint(8, 48)
        hi = min(hi, 2048)
    hi = max(hi, 4)
    lo = max(2, hi // rng.randint(1, 8)) if batch > 1 else hi
    return _case(None, op, w, layers, dec, vocab, lo, hi, batch, k, **more)


def _lengths(c):
    r = random.Random("%d %d %d" % (c["lo"], c["hi"], c["batch"]))
    return [r.randint(c["lo"], c["hi"]) for _ in range(c["batch"])]


# ----------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------
class _Shape:
    """The attributes that binding.make_config reads."""

    def __init__(self, c):
        self.n_layers, self.n_dec_layers, self.hidden = c["layers"], c["dec"], c["hidden"]
        self.n_heads, self.n_kv_heads, self.head_dim = c["heads"], c["kv_heads"], c["head_dim"]
        self.ffn, self.vocab, self.rope_base, self.rms_eps, self.dtype = c["ffn"], c["vocab"], c["rope_base"], EPS, c["dtype"]


def _weights(c, seed):
    """(name, tensor) of every weight, one at a time, on the GPU in the model's type."""
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + 17)
    h, q, kv, f = c["hidden"], c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"], c["ffn"]

    def normal(rows, cols, std):
        return (torch.randn(rows, cols, generator=g, device="cuda", dtype=torch.float32) * std).to(dt)

    def gain():
        return (1 + 0.1 * torch.randn(h, generator=g, device="cuda", dtype=torch.float32)).to(dt)

    deep = c["layers"] ** -0.5
    yield "embed", normal(c["vocab"], h, 0.02)
    yield "final_norm", gain()
    for i in range(c["layers"]):
        p = "layers.%d." % i
        yield p + "attn_norm", gain()
        yield p + "wq", normal(q, h, 0.02)
        yield p + "wk", normal(kv, h, 0.02)
        yield p + "wv", normal(kv, h, 0.02)
        yield p + "wo", normal(h, q, 0.003 * deep)
        yield p + "mlp_norm", gain()
        yield p + "w_gate", normal(f, h, 0.02)
        yield p + "w_up", normal(f, h, 0.02)
        yield p + "w_down", normal(h, f, 0.0005 * deep)


def _tokens(c, seed):
    """The prompts, and the tokens of the drafts or tree nodes."""
    r = np.random.default_rng([5, int(seed)])
    prompts = [r.integers(0, c["vocab"], n).astype(np.int32) for n in _lengths(c)]
    nodes = c.get("nodes", 0)
    drafts = r.integers(0, c["vocab"], nodes if nodes else c["batch"] * c["k"]).astype(np.int32)
    return prompts, drafts


def _parents(c):
    """A packed draft tree: the root, a chain of k nodes, then leaves spread over the root and the inner chain."""
    n, d = c["nodes"], c["k"]
    return np.array([-1] + list(range(d)) + [(i * 7) % d for i in range(n - 1 - d)], dtype=np.int32)


def prepare(case, seed):
    c, op = case, case["op"]
    prompts, drafts = _tokens(c, seed)
    rows = {"verify": c["batch"] * (c["k"] + 1), "prefill": c["batch"] * (c["k"] + 1), "draft": c["batch"] * c["k"],
            "tree": c.get("nodes", 0), "spec": c["hi"] - 1, "generate": c["batch"]}[op]
    extra = {"tree": c.get("nodes", 0) + 4, "generate": c.get("new", 0) + 2 * c["k"] + 4}.get(op, c["k"] + 4)
    draft = {"spec": 0, "tree": 0}.get(op, c["k"])
    dec = binding.Decoder(_Shape(c), max_batch=c["batch"], max_ctx=max(map(len, prompts)) + extra + draft + 2, max_draft=draft)
    code = binding.BF16 if c["dtype"] == "bf16" else binding.F32
    for name, t in _weights(c, seed):
        torch.cuda.synchronize()
        binding.seed_load_weights(dec.ctx, [(name, t.data_ptr(), code, True, tuple(t.shape))])
    s = dict(op=op, case=c, dec=dec, prompts=prompts, drafts=drafts)
    s["logits"] = torch.zeros(rows, c["vocab"], device="cuda", dtype=torch.float32)
    if op in ("verify", "tree"):
        out, _, _ = dec.generate(prompts, 0, 1)   # one token each: every sequence is then at its limit
    if op == "draft":
        dec.prefill(prompts)
    if op == "tree":
        s["parents"] = _parents(c)
        s["drafts"][0] = out[0][0]   # the root is the pending token
    if op == "spec":
        s["kv"] = torch.zeros(binding.seed_spec_kv_bytes(dec.cfg), device="cuda", dtype=torch.uint8)
        s["nll"] = torch.zeros(rows, device="cuda", dtype=torch.float32)
    torch.cuda.synchronize()
    return s


def run(s):
    c, dec, lg = s["case"], s["dec"], s["logits"]
    k, b, op = c["k"], c["batch"], s["op"]
    if op == "verify":
        binding.seed_verify(dec.ctx, k, b, s["drafts"] if k else None, lg.data_ptr())
        return lg
    if op == "tree":
        binding.seed_verify_tree(dec.ctx, s["drafts"], s["parents"], lg.data_ptr())
        return lg
    if op == "draft":
        return {"drafts": binding.seed_draft(dec.ctx, k, b, lg.data_ptr()), "logits": lg}
    if op == "prefill":
        binding.seed_prefill(dec.ctx, s["prompts"])
        binding.seed_verify(dec.ctx, k, b, s["drafts"] if k else None, lg.data_ptr())
        return lg
    if op == "spec":
        binding.seed_spec_forward(dec.ctx, s["prompts"][0], c["block"], s["kv"].data_ptr(), lg.data_ptr(), s["nll"].data_ptr())
        return {"logits": lg, "nll": s["nll"]}
    out, counts, _ = dec.generate(s["prompts"], k, c["new"], use_graph=True)
    binding.seed_draft(dec.ctx, 1, b, lg.data_ptr())
    return {"tokens": out, "logits": lg}


# ----------------------------------------------------------------------------------------------
# cost
# ----------------------------------------------------------------------------------------------
def _pass(c, layers, rows, keys, attended, head_rows):
    """Bytes and operations of one pass: `rows` rows through `layers` layers, `keys` cached positions read and `attended`
    (row, position) pairs of each layer, logits of `head_rows` rows."""
    es = 2 if c["dtype"] == "bf16" else 4
    h, q, kv, f = c["hidden"], c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"], c["ffn"]
    params = h * (2 * q + 2 * kv + 3 * f)
    nbytes = layers * (params * es + (keys + 2 * rows) * 2 * kv * es) + rows * h * es
    flops = layers * (2.0 * rows * params + 4.0 * attended * q)
    if head_rows:
        nbytes += c["vocab"] * h * es + head_rows * c["vocab"] * 4
        flops += 2.0 * head_rows * c["vocab"] * h
    return np.array([nbytes, flops], dtype=np.float64)


def work(case):
    c, op = case, case["op"]
    lens, b, k = _lengths(c), c["batch"], c["k"]
    tot = np.zeros(2)

    def verify(lens, rows, head=True):
        return _pass(c, c["layers"], rows * len(lens), sum(lens), sum(rows * (n + (rows + 1) / 2) for n in lens), rows * len(lens) if head else 0)

    def fill(layers):   # the prompts' weights once: one pass over all rows
        return _pass(c, layers, sum(n - 1 for n in lens), 0, sum((n - 1) * n / 2 for n in lens), 0)

    def step():
        return _pass(c, c["dec"], b, sum(lens), sum(lens), b)

    if op == "verify":
        tot += verify(lens, k + 1)
    elif op == "tree":
        tot += verify(lens, c["nodes"])
    elif op == "draft":
        tot += k * step()
    elif op == "prefill":
        tot += fill(c["layers"]) + verify([n - 1 for n in lens], k + 1)
    elif op == "spec":
        tot += fill(c["layers"]) + fill(c["dec"]) + _pass(c, 0, 0, 0, 0, lens[0] - 1)
    else:
        rounds = -(-c["new"] // (k + 1))
        tot += fill(c["layers"]) + rounds * (k * step() + verify(lens, k + 1)) + step()
        # logits stay inside the library in the rounds
        tot[0] -= rounds * b * (2 * k + 1) * c["vocab"] * 4
    return {"bytes": float(tot[0]), "flops": float(tot[1])}


def tolerance(case):
    # bf16 models: a key or value on the edge between two bf16 numbers may round either way, which travels through the
    # layers that follow (measured against 64 bits: up to 2e-4 over 4 layers, 5.5e-4 over 36); fp32 models: sums in
    # another order (measured: up to 6e-7)
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-4, "differ": 0.0}
    return {"rel": 2e-3 if case["layers"] > 4 else 8e-4, "max": 2e-2, "differ": 0.0}


# ----------------------------------------------------------------------------------------------
# the exact result: the same model in 64 bits, keys and values rounded as the cache stores them
# ----------------------------------------------------------------------------------------------
class _Exact:
    def __init__(self, c, seed):
        self.c = c
        self.w = dict(_weights(c, seed))
        self.cache = {}     # (sequence, layer) -> keys, values [positions, kv_heads, head_dim]

    def up(self, name):
        return self.w[name].double()

    def norm(self, x, name):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * self.up(name)

    def rope(self, x, pos):
        half = self.c["head_dim"] // 2
        inv = float(self.c["rope_base"]) ** (-torch.arange(half, device="cuda", dtype=torch.float64) * 2 / self.c["head_dim"])
        ang = pos.double()[:, None] * inv[None]
        co, si = ang.cos()[:, None], ang.sin()[:, None]
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * co - b * si, b * co + a * si], -1)

    def stored(self, x):
        return x.float().bfloat16().double() if self.c["dtype"] == "bf16" else x

    def embed(self, tokens):
        return self.w["embed"][torch.as_tensor(np.asarray(tokens), device="cuda").long()].double()

    def attend(self, q, keys, vals, allowed):
        """q [R, heads, d] over keys/vals [P, kv, d]; allowed(r0, r1) -> [r1 - r0, P] or one per source."""
        c = self.c
        g = c["heads"] // c["kv_heads"]
        out = torch.empty_like(q)
        step = max(1, (1 << 27) // (g * keys.shape[0]))
        for h in range(c["kv_heads"]):
            kt, v = keys[:, h].t().contiguous(), vals[:, h].contiguous()
            for r0 in range(0, q.shape[0], step):
                r1 = min(q.shape[0], r0 + step)
                s = torch.matmul(q[r0:r1, h * g:(h + 1) * g].reshape(-1, c["head_dim"]), kt) / math.sqrt(c["head_dim"])
                s = s.reshape(r1 - r0, g, -1).masked_fill(~allowed(r0, r1)[:, None], -math.inf).softmax(-1)
                out[r0:r1, h * g:(h + 1) * g] = torch.matmul(s.reshape(-1, s.shape[-1]), v).reshape(r1 - r0, g, -1)
        return out

    def layer(self, i, x, pos, attend):
        """attend(q, keys, values of these rows) -> attention output."""
        c, p = self.c, "layers.%d." % i
        a = self.norm(x, p + "attn_norm")
        heads = lambda n, cnt: (a @ self.up(p + n).t()).reshape(len(x), cnt, c["head_dim"])  # noqa: E731
        q, k = self.rope(heads("wq", c["heads"]), pos), self.stored(self.rope(heads("wk", c["kv_heads"]), pos))
        v = self.stored(heads("wv", c["kv_heads"]))
        x = x + attend(q, k, v).reshape(len(x), -1) @ self.up(p + "wo").t()
        a = self.norm(x, p + "mlp_norm")
        m = torch.nn.functional.silu(a @ self.up(p + "w_gate").t()) * (a @ self.up(p + "w_up").t())
        return x + m @ self.up(p + "w_down").t()

    def causal(self, seq, i, first, keep):
        """Attention of consecutive rows from position `first` over the cache below them and themselves."""
        def f(q, k, v):
            if (seq, i) in self.cache:
                ck, cv = self.cache[seq, i]
                k, v = torch.cat([ck[:first], k]), torch.cat([cv[:first], v])
            if keep:
                self.cache[seq, i] = (k, v)
            at = torch.arange(k.shape[0], device="cuda")
            return self.attend(q, k, v, lambda r0, r1: at[None] <= first + torch.arange(r0, r1, device="cuda")[:, None])
        return f

    def rows(self, seq, tokens, first, l0=0, keep=True):
        """Hidden states of consecutive tokens from position `first` through layers l0.., which the cache then holds."""
        x, pos = self.embed(tokens), first + torch.arange(len(tokens), device="cuda")
        for i in range(l0, self.c["layers"]):
            x = self.layer(i, x, pos, self.causal(seq, i, first, keep))
        return x

    def head(self, x):
        x, out = self.norm(x, "final_norm"), []
        for e in self.w["embed"].split(16384):
            out.append(x @ e.double().t())
        return torch.cat(out, -1)

    def draft(self, seq, token, first, steps):
        l0, toks, out = self.c["layers"] - self.c["dec"], [token], []
        for j in range(steps):
            out.append(self.head(self.rows(seq, toks[-1:], first + j, l0)))
            toks.append(int(out[-1].argmax()))
        return toks, torch.cat(out) if out else None

    def tree(self, tokens, parents, first):
        """Node rows: the cache below `first` and each node's ancestors."""
        n = len(tokens)
        depth, see = [0] * n, torch.eye(n, device="cuda", dtype=torch.bool)
        for i in range(1, n):
            depth[i] = depth[parents[i]] + 1
            see[i] |= see[parents[i]]
        x, pos = self.embed(tokens), first + torch.tensor(depth, device="cuda")
        allowed = torch.cat([torch.ones(n, first, device="cuda", dtype=torch.bool), see], 1)
        for i in range(self.c["layers"]):
            ck, cv = self.cache[0, i]
            x = self.layer(i, x, pos, lambda q, k, v: self.attend(
                q, torch.cat([ck[:first], k]), torch.cat([cv[:first], v]), lambda r0, r1: allowed[r0:r1]))
        return self.head(x)

    def spec(self, tokens, block):
        """Decoder rows over raw embeddings: a block's own rows causally, the deep cache below the block's start."""
        c = self.c
        n = len(tokens) - 1
        x, at = self.embed(tokens[:n]), torch.arange(n, device="cuda")
        start = at // block * block
        deep, own = at[None] < start[:, None], (at[None] >= start[:, None]) & (at[None] <= at[:, None])
        allowed = torch.cat([deep, own], 1)
        for i in range(c["layers"] - c["dec"], c["layers"]):
            ck, cv = self.cache[0, i]
            x = self.layer(i, x, at, lambda q, k, v: self.attend(
                q, torch.cat([ck[:n], k]), torch.cat([cv[:n], v]), lambda r0, r1: allowed[r0:r1]))
        return x


def exact(case, seed):
    c, op = case, case["op"]
    k, n_seq = c["k"], c["batch"]
    m = _Exact(c, seed)
    prompts, drafts = _tokens(c, seed)
    for b, p in enumerate(prompts):
        if len(p) > 1:
            m.rows(b, p[:-1], 0)
    if op in ("verify", "prefill"):
        out = []
        for b, p in enumerate(prompts):
            first, tok = len(p) - 1, int(p[-1])
            if op == "verify":
                tok = int(m.head(m.rows(b, [tok], first)).argmax())
                first += 1
            out.append(m.head(m.rows(b, [tok] + [int(t) for t in drafts[b * k:(b + 1) * k]], first, keep=False)))
        return torch.cat(out)
    if op == "tree":
        p = prompts[0]
        drafts[0] = int(m.head(m.rows(0, p[-1:], len(p) - 1)).argmax())
        return m.tree([int(t) for t in drafts], list(_parents(c)), len(p))
    if op == "draft":
        got = [m.draft(b, int(p[-1]), len(p) - 1, k) for b, p in enumerate(prompts)]
        return {"drafts": np.array([t[1:] for t, _ in got], dtype=np.int32), "logits": torch.cat([x for _, x in got])}
    if op == "spec":
        x = m.spec(prompts[0], c["block"])
        logits, nll = [], []
        for r in range(0, len(x), 128):
            y = m.head(x[r:r + 128])
            t = torch.as_tensor(prompts[0][r + 1:r + 1 + len(y)], device="cuda").long()
            nll.append(torch.logsumexp(y, -1) - y.gather(1, t[:, None])[:, 0])
            logits.append(y)
        return {"logits": torch.cat(logits), "nll": torch.cat(nll)}
    tokens, logits = np.full((n_seq, c["new"]), -1, dtype=np.int32), []
    done = {}
    for b, p in enumerate(prompts):
        text = [int(t) for t in p]
        while len(text) < len(p) + c["new"]:
            first = len(text) - 1
            toks, _ = m.draft(b, text[-1], first, k) if k else ([text[-1]], None)
            best = m.head(m.rows(b, toks, first)).argmax(-1).tolist()
            a = 0
            while a < k and best[a] == toks[a + 1]:
                a += 1
            text += best[:a + 1]
        tokens[b] = text[len(p):len(p) + c["new"]]
        done[b] = text
    for b, text in done.items():
        logits.append(m.draft(b, text[-1], len(text) - 1, 1)[1])
    return {"tokens": tokens, "logits": torch.cat(logits)}
