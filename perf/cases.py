"""The work that programs have this library do, as cases that can be timed and checked.

Four kinds, all through the package's public calls on the current stream:

    block     one decode step of one decoder block       cfpp_block_decode / cfpp_block_decode_static
    stack     one decode step of a stack of blocks       cfpp_stack_replay of a captured step
    generate  one token with logits, call by call        cfpp_lm_embed, cfpp_stack_decode, cfpp_lm_next
    prefill   a prompt (or a part of one)                cfpp_stack_prefill_gemm / cfpp_stack_prefill

A case holds plain values only.  Everything a program would keep (packed weights, caches,
workspace, scratch, the captured graph) is made by prepare() from the seed; run() is one pass
and returns the outputs together with views of the cache rows that the pass appended.
exact() computes the same outputs with torch in 64 bits; what later tokens read of an appended
row is rounded to fp16 there as well, because the cache stores fp16.
"""
import math
import random

import torch

import paper_2604_23553_amd as cf

# name: hidden, heads, head size, rotated dimensions, MLP width
SHAPES = {
    "h512": (512, 8, 64, 16, 2048),
    "h1024": (1024, 8, 128, 32, 4096),
    "h1280": (1280, 16, 80, 20, 5120),
    "h1536": (1536, 24, 64, 16, 6144),
    "h2560": (2560, 32, 80, 20, 10240),        # the Pythia-2.8B shape, 32 layers
    "h4096": (4096, 32, 128, 32, 16384),       # the Pythia-6.9B shape, 32 layers
}
VOCAB = 50304
ROPE_BASE, LN_EPS = 10000.0, 1e-5
TANH_GELU, SEQUENTIAL_RESIDUAL = 1, 2          # cfpp_config.flags
MOST_FLOPS = 41e12                             # a pass of the largest listed case
TENSORS = ("ln1_g", "ln1_b", "ln2_g", "ln2_b", "w_qkv", "b_qkv", "w_dense", "b_dense", "w_up", "b_up", "w_down", "b_down")


def _case(kind, shape, layers=1, batch=1, lo=0, hi=0, cap=0, tokens=0, pos0=0, rows=0, call="", flags=0, **more):
    """lo, hi: cached positions of a decode step's sequences; cap: positions the cache holds;
    tokens, pos0, rows: of a prompt, its first position and the tokens per pass (0: groups of 8)."""
    return dict(more, kind=kind, shape=shape, layers=layers, batch=batch, lo=lo, hi=hi, cap=cap, tokens=tokens, pos0=pos0,
                rows=rows, call=call, flags=flags)


def listed():
    return [
        # the smallest call: a small model's block, a short context; launches and latency
        _case("block", "h512", lo=128, hi=128, cap=256, name="block_h512_s128"),
        # one block on its own, as a pipeline stage or a host-driven loop calls it
        _case("block", "h2560", lo=1024, hi=1024, cap=1088, name="block_h2560_s1024"),
        # a serving step of one layer for a full group of sequences of very different lengths
        _case("block", "h4096", batch=8, lo=1024, hi=8192, cap=8256, name="block_h4096_b8"),
        # the token loop: a 32-layer model, long context, one sequence
        _case("stack", "h2560", layers=32, lo=4096, hi=4096, cap=4160, name="stack_h2560_s4096"),
        # the same for the larger model, an odd context length
        _case("stack", "h4096", layers=32, lo=1777, hi=1777, cap=2048, name="stack_h4096_s1777"),
        # a serving step of a stage of 12 layers, five sequences of short to middling length
        _case("stack", "h2560", layers=12, batch=5, lo=37, hi=2048, cap=2112, name="stack_h2560_b5"),
        # a generated token with its logits, called step by step (sampling on the host needs them)
        _case("generate", "h2560", layers=32, lo=300, hi=300, cap=1024, name="generate_h2560_s300"),
        # a short instruction as the first prompt
        _case("prefill", "h2560", layers=32, tokens=37, rows=128, cap=1024, name="prefill_h2560_t37"),
        # the benchmark's prompt
        _case("prefill", "h2560", layers=32, tokens=512, rows=512, cap=1024, name="prefill_h2560_t512"),
        # a later part of a long prompt through a stage of the larger model: odd length, cached context, the GELU option
        _case("prefill", "h4096", layers=4, tokens=1531, pos0=700, rows=1536, cap=4096, flags=TANH_GELU, name="prefill_h4096_t1531"),
        # the longest pass
        _case("prefill", "h2560", layers=16, tokens=4096, rows=4096, cap=4160, name="prefill_h2560_t4096"),
        # a few tokens appended to a running conversation, without scratch memory
        _case("prefill", "h2560", layers=32, batch=8, tokens=8, pos0=1000, cap=1088, name="prefill_h2560_t8_groups"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["block", "block", "stack", "stack", "generate", "prefill", "prefill", "prefill", "prefill"])
    shape = rng.choice(["h512", "h1024", "h1280", "h1536", "h2560", "h2560", "h2560", "h4096", "h4096", "h4096"])
    flags = rng.choice([0, 0, 0, TANH_GELU])
    if kind == "prefill":
        if rng.random() < 0.2:
            c = _case(kind, shape, layers=_log_int(rng, 1, 32), batch=8, tokens=_log_int(rng, 1, 64), pos0=_log_int(rng, 1, 4000) - 1, flags=flags)
        else:
            tokens = _log_int(rng, 1, 4096)
            rows = -(-tokens // 128) * 128
            if tokens > 256 and rng.random() < 0.25:
                rows = rng.choice([128, 256, 512])          # a long prompt in several passes
            pos0 = rng.choice([0, 0, rng.randrange(1, 4000)])
            c = _case(kind, shape, layers=_log_int(rng, 1, 32), tokens=tokens, pos0=pos0, rows=min(rows, 4096), flags=flags)
        c["cap"] = c["pos0"] + c["tokens"] + rng.randrange(0, 129)
        while work(c)["flops"] > MOST_FLOPS and c["layers"] > 1:
            c["layers"] -= 1
        return c
    hi = _log_int(rng, 16, 8192)
    if kind == "generate":
        c = _case(kind, shape, layers=_log_int(rng, 1, 24), lo=hi, hi=hi, flags=flags)
    else:
        batch = rng.choice([1, 1, 2, 3, 4, 5, 6, 7, 8])
        layers = 1 if kind == "block" else _log_int(rng, 2, 32)
        if layers * batch > 60:
            layers = 60 // batch
        c = _case(kind, shape, layers=layers, batch=batch, lo=hi if batch == 1 else rng.randrange(0, hi + 1), hi=hi, flags=flags)
        if kind == "block" and batch == 1:
            c["call"] = rng.choice(["", "", "static"])
            c["flags"] = rng.choice([0, 0, TANH_GELU, SEQUENTIAL_RESIDUAL])
    c["cap"] = c["hi"] + 1 + rng.randrange(0, 129)
    return c


def _lens(case):
    """Cached positions of each sequence: the longest is `hi`, the others anywhere in [lo, hi]."""
    r = random.Random(case["lo"] * 8209 + case["hi"] * 17 + case["batch"])
    n = [r.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]
    n[r.randrange(case["batch"])] = case["hi"]
    return n


def _gen(seed, what, layer=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + what * 4099 + layer * 31 + 7) & 0x7FFFFFFFFFFF)
    return g


def _normal(g, dims, std=1.0, mean=0.0):
    t = torch.randn(dims, generator=g, device="cuda", dtype=torch.float32)
    if std != 1.0:
        t.mul_(std)
    if mean:
        t.add_(mean)
    return t.half()


def _weights(case, seed, layer):
    """The 12 canonical fp16 tensors of a block: weights and biases N(0, 0.02), LayerNorm gains 1 + N(0, 0.02)."""
    h, H, d, r, f = SHAPES[case["shape"]]
    dims = {"ln1_g": (h,), "ln1_b": (h,), "ln2_g": (h,), "ln2_b": (h,), "w_qkv": (3 * h, h), "b_qkv": (3 * h,),
            "w_dense": (h, h), "b_dense": (h,), "w_up": (f, h), "b_up": (f,), "w_down": (h, f), "b_down": (h,)}
    g = _gen(seed, 1, layer)
    return {n: _normal(g, dims[n], 0.02, 1.0 if n in ("ln1_g", "ln2_g") else 0.0) for n in TENSORS}


def _cache(case, seed, layer):
    """A layer's cache as the library lays it out, [K, V][batch][head][d / 16][position][16], every slot N(0, 1)."""
    h, H, d, r, f = SHAPES[case["shape"]]
    return _normal(_gen(seed, 2, layer), (2, case["batch"], H, d // 16, case["cap"], 16))


def _head(case, seed):
    h = SHAPES[case["shape"]][0]
    g = _gen(seed, 3)
    return {"embed": _normal(g, (VOCAB, h)), "lnf_g": _normal(g, (h,), 0.02, 1.0), "lnf_b": _normal(g, (h,), 0.02),
            "w_lm": _normal(g, (VOCAB, h), 0.02)}


def _x(case, seed):
    n = case["tokens"] if case["kind"] == "prefill" else case["batch"]
    return _normal(_gen(seed, 4), (n, SHAPES[case["shape"]][0]))


def _tokens(case, seed):
    return torch.randint(0, VOCAB, (case["cap"] + 1,), generator=_gen(seed, 5), device="cuda", dtype=torch.int32)


def _config(case):
    h, H, d, r, f = SHAPES[case["shape"]]
    return cf.Config(h, H, d, r, f, case["layers"], case["cap"], case["batch"], ROPE_BASE, LN_EPS, case["flags"])


def _rows(case, caches):
    """Views of the cache rows that a pass appends."""
    if case["kind"] == "prefill":
        return [kv[:, 0, :, :, case["pos0"]:case["pos0"] + case["tokens"]] for kv in caches]
    return [kv[:, b, :, :, p] for kv in caches for b, p in enumerate(_lens(case))]


class _State:
    """What a program holds between calls; the library's context goes with it."""

    ctx = 0

    def __del__(self):
        if self.ctx:
            torch.cuda.synchronize()
            cf.cfpp_destroy(self.ctx)


def prepare(case, seed):
    s = _State()
    s.case, s.cfg = case, _config(case)
    s.packed, s.kv = [], []
    u8 = dict(dtype=torch.uint8, device="cuda")
    for l in range(case["layers"]):
        w = _weights(case, seed, l)
        p = torch.empty(cf.cfpp_packed_layer_bytes(s.cfg), **u8)
        cf.cfpp_pack_layer(s.cfg, w, p, torch.cuda.current_stream().cuda_stream)
        s.packed.append(p)
        s.kv.append(_cache(case, seed, l))
    nbytes = cf.cfpp_workspace_bytes(s.cfg)
    s.ws = torch.empty(nbytes, **u8)
    s.x = _x(case, seed)
    s.out = torch.zeros_like(s.x)
    s.rows = _rows(case, s.kv)
    if case["kind"] != "prefill":
        s.pos = torch.tensor(_lens(case), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    if case["call"] != "static":
        s.ctx = cf.cfpp_create(s.cfg, s.ws, nbytes)
    if case["kind"] == "generate":
        s.pos0 = s.pos.clone()
        s.head = _head(case, seed)
        s.lm = cf.Lm.of(s.head["embed"], s.head["lnf_g"], s.head["lnf_b"], s.head["w_lm"], VOCAB)
        s.tokens = _tokens(case, seed)
        s.logits = torch.zeros(VOCAB, dtype=torch.float32, device="cuda")
    elif case["kind"] == "stack":
        side = torch.cuda.Stream()
        torch.cuda.synchronize()
        cf.cfpp_stack_capture(s.ctx, s.packed, s.kv, s.x, s.pos, case["batch"], s.out, side.cuda_stream)
    elif case["kind"] == "prefill" and case["rows"]:
        s.scratch_bytes = cf.cfpp_prefill_scratch_bytes(s.cfg, case["rows"])
        s.scratch = torch.empty(s.scratch_bytes, **u8)
    torch.cuda.synchronize()
    return s


def run(s):
    c, stream = s.case, torch.cuda.current_stream().cuda_stream
    if c["kind"] == "block":
        if c["call"] == "static":
            cf.cfpp_block_decode_static(s.cfg, s.packed[0], s.kv[0], s.x, s.pos, c["batch"], s.out, stream)
        else:
            cf.cfpp_block_decode(s.ctx, s.packed[0], s.kv[0], s.x, s.pos, c["batch"], s.out, stream)
    elif c["kind"] == "stack":
        cf.cfpp_stack_replay(s.ctx, stream)
    elif c["kind"] == "generate":
        s.pos.copy_(s.pos0)                                # the request's position; the last call advances it
        cf.cfpp_lm_embed(s.ctx, s.lm, s.tokens, s.pos, s.x, stream)
        cf.cfpp_stack_decode(s.ctx, s.packed, s.kv, s.x, s.pos, 1, s.out, stream)
        cf.cfpp_lm_next(s.ctx, s.lm, s.out, s.tokens, s.pos, s.logits, stream)
        return {"logits": s.logits, "tokens": s.tokens, "pos": s.pos, "hidden": s.out, "rows": s.rows}
    elif c["rows"]:
        cf.cfpp_stack_prefill_gemm(s.ctx, s.packed, s.kv, s.x, c["pos0"], c["tokens"], 0, s.out, s.scratch, s.scratch_bytes,
                                   c["rows"], stream)
    else:
        cf.cfpp_stack_prefill(s.ctx, s.packed, s.kv, s.x, c["pos0"], c["tokens"], 0, s.out, stream)
    return {"out": s.out, "rows": s.rows}


def work(case):
    """Every parameter, cached row and input read once, every appended row and output written once; two operations a
    multiplication."""
    h, H, d, r, f = SHAPES[case["shape"]]
    params = 4 * h * h + 2 * h * f + 3 * h + h + f + h + 4 * h
    if case["kind"] == "prefill":
        n, cached = case["tokens"], case["pos0"]
        pairs = sum(range(cached + 1, cached + n + 1))
    else:
        lens = _lens(case)
        n, cached = len(lens), sum(lens)
        pairs = cached + n
    per_layer = 2 * params + 2 * 2 * h * (cached + n)
    flops = case["layers"] * (2 * n * (4 * h * h + 2 * h * f) + 4 * h * pairs)
    nbytes = case["layers"] * per_layer + 2 * 2 * n * h
    if case["kind"] == "generate":
        nbytes += 2 * (VOCAB * h + h + 2 * h) + 4 * VOCAB
        flops += 2 * VOCAB * h
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """fp16 results of sums in 32 bits: against exact() every path is 2.0e-4 to 2.4e-4 off (the rounding of the results),
    of which this is four times.  "max": an output or appended row next to a rounding boundary moves by one fp16 step
    (up to 1e-3 of it) under another order of the sums; in a stack such a step in one layer's row reaches the next."""
    tol = {"rel": 1e-3, "max": 2e-2 if case["layers"] > 1 else 4e-3}
    if case["kind"] == "generate":
        tol["differ"] = 2.0 / (case["cap"] + 1)            # two equal leaders among the logits, at most
    return tol


# ---- the same in 64 bits, by torch alone ------------------------------------------------
def _layer_norm(x, g, b):
    return torch.nn.functional.layer_norm(x, (x.shape[-1],), g.double(), b.double(), LN_EPS)


def _linear(x, w, b=None):
    y = x @ w.double().t().contiguous()
    return y if b is None else y + b.double()


def _rotate(v, pos, r):
    """v [n, H, d] at positions pos [n]: half-split pairs (i, i + r/2) of the first r dimensions."""
    if not r:
        return v
    theta = ROPE_BASE ** (-2.0 * torch.arange(r // 2, device="cuda", dtype=torch.float64) / r)
    ang = pos.double()[:, None, None] * theta
    a, b = v[..., :r // 2], v[..., r // 2:r]
    return torch.cat([a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos(), v[..., r:]], -1)


def _attend(q, k, v, pos):
    """q [n, H, d] at positions pos [n] over k, v [H, S, d]: row i sees positions <= pos[i]."""
    out = torch.empty_like(q)
    S = k.shape[1]
    for a in range(0, q.shape[0], 512):
        qq = q[a:a + 512].transpose(0, 1).contiguous()
        s = torch.matmul(qq, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
        late = torch.arange(S, device="cuda")[None, :] > pos[a:a + 512, None]
        s.masked_fill_(late[None], -math.inf)
        out[a:a + 512] = torch.matmul(torch.softmax(s, -1), v).transpose(0, 1)
    return out


def _gelu(z, flags):
    return torch.nn.functional.gelu(z, approximate="tanh" if flags & TANH_GELU else "none")


def _block(case, w, kv, x, pos, seq):
    """x [n, h] through one block; row i is position pos[i] of sequence seq[i]; kv (library layout) gets the new rows.
    Returns the block's output and the new rows before their rounding, [2, n, H, d / 16, 16]."""
    h, H, d, r, f = SHAPES[case["shape"]]
    n = x.shape[0]
    qkv = _linear(_layer_norm(x, w["ln1_g"], w["ln1_b"]), w["w_qkv"], w["b_qkv"]).view(n, H, 3, d)
    q = _rotate(qkv[:, :, 0], pos, r)
    k = _rotate(qkv[:, :, 1], pos, r)
    unrounded = torch.stack([k, qkv[:, :, 2]]).view(2, n, H, d // 16, 16)
    new = unrounded.half()
    att = torch.empty_like(q)
    for b in sorted(set(seq)):
        at = [i for i, t in enumerate(seq) if t == b]
        lo, hi = at[0], at[-1] + 1                         # (a sequence's rows are consecutive)
        p = pos[lo:hi]
        kv[:, b, :, :, p] = new[:, lo:hi].permute(0, 2, 3, 1, 4)
        S = int(p.max()) + 1
        full = kv[:, b, :, :, :S].permute(0, 1, 3, 2, 4).reshape(2, H, S, d).double()
        att[lo:hi] = _attend(q[lo:hi], full[0], full[1], p)
    a = _linear(att.reshape(n, h), w["w_dense"], w["b_dense"])
    base = x + a if case["flags"] & SEQUENTIAL_RESIDUAL else x
    m = _gelu(_linear(_layer_norm(base, w["ln2_g"], w["ln2_b"]), w["w_up"], w["b_up"]), case["flags"])
    return x + a + _linear(m, w["w_down"], w["b_down"]), unrounded


def exact(case, seed):
    if case["kind"] == "prefill":
        n = case["tokens"]
        pos, seq = torch.arange(case["pos0"], case["pos0"] + n, device="cuda"), [0] * n
    else:
        pos, seq = torch.tensor(_lens(case), device="cuda"), list(range(case["batch"]))
    if case["kind"] == "generate":
        head, tokens = _head(case, seed), _tokens(case, seed)
        x = head["embed"][int(tokens[case["hi"]])][None].double()
    else:
        x = _x(case, seed).double()
    rows = []
    for l in range(case["layers"]):
        x, new = _block(case, _weights(case, seed, l), _cache(case, seed, l), x, pos, seq)
        rows += [new.permute(0, 2, 3, 1, 4)] if case["kind"] == "prefill" else [new[:, b] for b in range(case["batch"])]
    if case["kind"] == "generate":
        logits = _linear(_layer_norm(x, head["lnf_g"], head["lnf_b"]), head["w_lm"])[0]
        return {"logits": logits, "tokens": None, "pos": None, "hidden": x, "rows": rows}
    return {"out": x, "rows": rows}
