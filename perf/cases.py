"""Timed cases of the decode-step library: what a serving instance has it do, through the public binding.

A case is a dict of plain values.  `listed()` names the standing ones, `draw(rng)` gives another of the same ranges,
`prepare(case, seed)` makes what the program holds before the call, `run(state)` is one pass, `work(case)` the bytes
and operations the pass cannot do without, `tolerance(case)` how far two correct implementations may be apart, and
`exact(case, seed)` the same result in 64 bits, written in plain torch.

Kinds of case
  step       one decode step (q_len > 1: one multi-token verify step) of a Llama-style decoder over a paged cache
  attention  paged grouped-query attention of one layer
  ffn        one SwiGLU feed-forward block
  linear     one plain projection
  prefill    one layer's K/V of a few requests written to their pages, and read back in token order
  swap       one request's pages moved to pinned host memory and restored into other pages
"""
import math

import numpy as np
import torch

from paper_2501_08090_amd import binding as B
from paper_2501_08090_amd import inputs as I

PAGE = 16
CHUNK = 1 << 17  # tokens of synthetic cache made at a time
POOL_OUT = 160 << 20  # a step's cache that can never grow beyond this is returned beside the logits

SHAPES = {"tiny": I.TINY, "8b": I.LLAMA_8B, "70b": I.LLAMA_70B}


def _shape(name, **over):
    m = SHAPES[name]
    c = {k: m[k] for k in ("hidden", "n_q_heads", "n_kv_heads", "head_dim", "ffn", "vocab", "rope_base")}
    c.update(over)
    return c


def _heads(c):
    return {k: c[k] for k in ("n_q_heads", "n_kv_heads", "head_dim")}


def _lens(kind, median, lo, hi):
    return {"lens": kind, "median": median, "lo": lo, "hi": hi}


def listed():
    eight = _shape("8b")
    return [
        # the smallest call: a toy decoder, four requests; nothing but launches and latency
        dict(name="step_tiny_b4", kind="step", layers=2, batch=4, q_len=1, **_shape("tiny"), **_lens("uniform", 0, 16, 128)),
        # one interactive user on an 8B-wide decoder (four of its layers and the head): the weight stream at one row
        dict(name="step_8b_b1", kind="step", layers=4, batch=1, q_len=1, **eight, **_lens("lognormal", 512, 16, 8192)),
        # a lightly loaded instance, an odd number of requests of both classes
        dict(name="step_8b_b11_mixed", kind="step", layers=4, batch=11, q_len=1, **eight, **_lens("mixed", 512, 16, 8192)),
        # the benchmark's batch and context population
        dict(name="step_8b_b64", kind="step", layers=4, batch=64, q_len=1, **eight, **_lens("lognormal", 800, 64, 4096)),
        # a batch-class instance near the batch size its autoscaler climbs to, both classes of request
        dict(name="step_8b_b500_mixed", kind="step", layers=2, batch=500, q_len=1, **eight, **_lens("mixed", 512, 16, 8192)),
        # speculative decoding: 32 requests verify four drafted tokens each
        dict(name="verify_8b_b32x4", kind="step", layers=4, batch=32, q_len=4, **eight, **_lens("lognormal", 800, 64, 4096)),
        # long documents: attention over 24k..32k tokens for 32 requests
        dict(name="attn_8b_b32_long", kind="attention", batch=32, **_heads(eight), **_lens("uniform", 0, 24576, 32768)),
        # attention of a large ragged batch
        dict(name="attn_8b_b512_mixed", kind="attention", batch=512, **_heads(eight), **_lens("mixed", 512, 16, 8192)),
        # the feed-forward block of a 70B-wide layer at a batch between the tile sizes
        dict(name="ffn_70b_r100", kind="ffn", rows=100, hidden=8192, ffn=28672),
        # the feed-forward block of an 8B-wide layer at the batch sizes of batch-class instances
        dict(name="ffn_8b_r2048", kind="ffn", rows=2048, hidden=4096, ffn=14336),
        # three prompts enter the cache of one layer and are read back
        dict(name="prefill_8b_3x2711", kind="prefill", requests=3, tokens=2711, n_kv_heads=8, head_dim=128),
        # an interactive request evicts a batch one: 517 tokens, all 32 layers, out to the host and back
        dict(name="swap_8b_517", kind="swap", layers=32, tokens=517, n_kv_heads=8, head_dim=128),
    ]


def _log(rng, lo, hi):
    """a whole number, spread evenly over the logarithm of the range"""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("step",) * 6 + ("attention",) * 2 + ("ffn",) * 2 + ("linear", "prefill", "swap"))
    if kind == "step":
        if rng.random() < 0.5:
            c = _shape("8b")
        else:  # any Llama-style decoder
            d = rng.choice((64, 128))
            n_kv = rng.choice((1, 2, 4, 8))
            c = dict(hidden=16 * _log(rng, 16, 320), n_q_heads=n_kv * rng.choice((1, 2, 4, 8)), n_kv_heads=n_kv, head_dim=d,
                     ffn=16 * _log(rng, 43, 1000), vocab=_log(rng, 1000, 128256), rope_base=rng.choice((10000.0, 500000.0)))
        q_len = rng.choice((1, 1, 1, 1, 2, 3, 4, 5))
        batch = _log(rng, 1, 500 // q_len)
        lens = rng.choice((_lens("lognormal", _log(rng, 100, 1500), 16, 8192), _lens("uniform", 0, 0, _log(rng, 64, 4000)),
                           _lens("mixed", 512, 16, 8192)))
        return dict(kind="step", layers=rng.randint(1, 2), batch=batch, q_len=q_len, **c, **lens)
    if kind == "attention":
        d = rng.choice((64, 128, 128))
        n_kv = rng.choice((2, 4, 8, 8))
        g = rng.choice((1, 4, 4, 8))
        if rng.random() < 0.3:
            return dict(kind=kind, batch=rng.randint(1, 32), n_q_heads=n_kv * g, n_kv_heads=n_kv, head_dim=d, **_lens("uniform", 0, 8192, 32768))
        return dict(kind=kind, batch=_log(rng, 1, 512), n_q_heads=n_kv * g, n_kv_heads=n_kv, head_dim=d,
                    **rng.choice((_lens("lognormal", _log(rng, 100, 2000), 16, 8192), _lens("mixed", 512, 16, 8192))))
    if kind == "ffn":
        return dict(kind=kind, rows=_log(rng, 1, 2048), hidden=16 * _log(rng, 16, 256), ffn=16 * _log(rng, 43, 896))
    if kind == "linear":
        return dict(kind=kind, rows=_log(rng, 1, 1024), n=_log(rng, 500, 30000), k=16 * _log(rng, 16, 512))
    if kind == "prefill":
        return dict(kind=kind, requests=rng.randint(1, 4), tokens=_log(rng, 17, 2700), n_kv_heads=rng.choice((1, 2, 8)), head_dim=rng.choice((64, 128)))
    return dict(kind="swap", layers=_log(rng, 2, 32), tokens=_log(rng, 16, 517), n_kv_heads=rng.choice((2, 8)), head_dim=rng.choice((64, 128)))


# ---- inputs, made from the seed alone --------------------------------------------------------------------------

def _number(*names):
    h = 1469598103934665603
    for ch in "/".join(str(n) for n in names).encode():
        h = (h ^ ch) * 1099511628211 & 0x7FFFFFFFFFFFFFFF
    return h


def _normal(shape, std, *names, dtype=torch.bfloat16, mean=0.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(_number(*names))
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=g)


def _context(c, seed):
    """tokens already cached for each request"""
    n = c["batch"]
    rng = np.random.default_rng(_number("lens", seed))
    if c["lens"] == "uniform":
        return rng.integers(c["lo"], c["hi"] + 1, n).astype(np.int32)
    got = np.clip(np.rint(c["median"] * np.exp(0.8 * rng.standard_normal(n))), c["lo"], c["hi"])
    if c["lens"] == "mixed":  # three in ten are batch-class requests with long contexts
        got = np.where(np.isin(np.arange(n) % 10, (3, 6, 9)), rng.integers(c["hi"] // 4, c["hi"] + 1, n), got)
    return got.astype(np.int32)


def _mean_context(c):
    """expected tokens per request, from the distribution (the lengths themselves depend on the seed)"""
    if c["lens"] == "uniform":
        return 0.5 * (c["lo"] + c["hi"])
    m = min(c["median"] * math.exp(0.32), c["hi"])
    return 0.7 * m + 0.3 * 0.625 * c["hi"] if c["lens"] == "mixed" else m


def _table(lens, new, seed):
    """shuffled pages with room for `new` more tokens of each request, -1 in unused entries; pages in the pool"""
    need = (lens.astype(np.int64) + new + PAGE - 1) // PAGE
    total = int(need.sum())
    pool = total + total // 7 + 1
    ids = np.random.default_rng(_number("pages", seed)).permutation(pool)[:total].astype(np.int32)
    bt = np.full((len(lens), int(need.max())), -1, np.int32)
    at = 0
    for i, k in enumerate(need):
        bt[i, :k] = ids[at:at + k]
        at += k
    return bt, pool


def _layer(c, seed, l):
    H, F, d = c["hidden"], c["ffn"], c["head_dim"]
    qn, kn = c["n_q_heads"] * d, c["n_kv_heads"] * d
    w = {n: _normal(s, 0.02, seed, n, l) for n, s in dict(wq=(qn, H), wk=(kn, H), wv=(kn, H), wo=(H, qn), w_gate=(F, H), w_up=(F, H), w_down=(H, F)).items()}
    for n in ("attn_norm", "ffn_norm"):
        w[n] = _normal((H,), 0.1, seed, n, l, mean=1.0)
    return w


def _head(c, seed):
    return dict(embed=_normal((c["vocab"], c["hidden"]), 0.02, seed, "embed"), final_norm=_normal((c["hidden"],), 0.1, seed, "final", mean=1.0),
                lm_head=_normal((c["vocab"], c["hidden"]), 0.02, seed, "lm_head"))


def _cache(c, total, seed, l, at):
    """K and V of the cached tokens at .. at + CHUNK of one layer, request after request"""
    shape = (min(CHUNK, total - at), c["n_kv_heads"], c["head_dim"])
    return _normal(shape, 1.0, seed, "k", l, at), _normal(shape, 1.0, seed, "v", l, at)


def _tokens(c, seed):
    return np.random.default_rng(_number("tokens", seed)).integers(0, c["vocab"], (c["batch"], c["q_len"])).astype(np.int32)


def _fill(pool, c, lens, bt, layers, seed):
    seq, pos = (torch.from_numpy(a).cuda() for a in I.prefill_index(lens))
    total = int(lens.sum())
    for l in range(layers):
        for at in range(0, total, CHUNK):
            k, v = _cache(c, total, seed, l, at)
            pool.append(l, k, v, bt, seq[at:at + CHUNK].contiguous(), pos[at:at + CHUNK].contiguous())


def _pool(model, pages):
    return B.KVPool(model, memory=torch.zeros(pages * model.kv_block_bytes(), dtype=torch.uint8, device="cuda"))


def _bare_model(c, layers, max_batch, max_blocks):
    """a model that only lends its cache geometry and attention workspace"""
    m = dict(n_layers=layers, hidden=256, n_q_heads=c.get("n_q_heads", c["n_kv_heads"]), n_kv_heads=c["n_kv_heads"], head_dim=c["head_dim"], ffn=16, vocab=16,
             rope_base=500000.0, rms_eps=1e-5)
    return B.Model(m, max_batch, max_blocks)


# ---- the program's side ----------------------------------------------------------------------------------------

def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"kind": kind}
    if kind == "step":
        lens = _context(c, seed)
        bt, pages = _table(lens, c["q_len"], seed)
        m = dict({k: c[k] for k in ("hidden", "n_q_heads", "n_kv_heads", "head_dim", "ffn", "vocab", "rope_base")}, n_layers=c["layers"], rms_eps=1e-5)
        model = B.Model(m, c["batch"] * c["q_len"], bt.shape[1])
        for l in range(c["layers"]):
            model.load_layer(l, **_layer(c, seed, l))
        model.load_head(**_head(c, seed))
        most = c["batch"] * ((c["hi"] + c["q_len"] + PAGE - 1) // PAGE + 1)  # pages, whatever the seed
        small = most * model.kv_block_bytes() <= POOL_OUT
        pool = _pool(model, most if small else pages)
        bt = torch.from_numpy(bt).cuda()
        _fill(pool, c, lens, bt, c["layers"], seed)
        tok = torch.from_numpy(_tokens(c, seed)).cuda()
        s.update(model=model, pool=pool, bt=bt, lens=torch.from_numpy(lens).cuda(), tok=tok if c["q_len"] > 1 else tok.view(-1),
                 q_len=c["q_len"], logits=torch.zeros((c["batch"], c["q_len"], c["vocab"]) if c["q_len"] > 1 else (c["batch"], c["vocab"]), device="cuda"),
                 cache=pool.memory.view(torch.bfloat16) if small else None)
    elif kind == "attention":
        lens = np.maximum(_context(c, seed), 1)
        bt, pages = _table(lens, 0, seed)
        model = _bare_model(c, 1, c["batch"], bt.shape[1])
        pool = _pool(model, pages)
        bt = torch.from_numpy(bt).cuda()
        _fill(pool, c, lens, bt, 1, seed)
        s.update(model=model, pool=pool, bt=bt, lens=torch.from_numpy(lens).cuda(), q=_q(c, seed))
    elif kind == "ffn":
        wg, wu, wd, x = _ffn(c, seed)
        s.update(gate_up=B.GateUp(wg, wu), down=B.Linear(wd), x=x)
        torch.cuda.synchronize()
    elif kind == "linear":
        w, x = _linear(c, seed)
        s.update(w=B.Linear(w), x=x)
        torch.cuda.synchronize()
    elif kind == "prefill":
        lens = np.full(c["requests"], c["tokens"], np.int32)
        bt, pages = _table(lens, 1, seed)
        model = _bare_model(c, 1, c["requests"], bt.shape[1])
        seq, pos = I.prefill_index(lens)
        k, v = _prompt(c, seed)
        s.update(model=model, pool=_pool(model, pages), bt=torch.from_numpy(bt).cuda(), n=c["tokens"], k=k, v=v, seq=torch.from_numpy(seq).cuda(), pos=torch.from_numpy(pos).cuda())
    else:
        lens = np.array([c["tokens"], c["tokens"]], np.int32)  # the request's pages, and those it restarts in
        bt, pages = _table(lens, 1, seed)
        model = _bare_model(c, c["layers"], 2, bt.shape[1])
        pool = _pool(model, pages)
        bt = torch.from_numpy(bt).cuda()
        _fill(pool, c, lens[:1], bt, c["layers"], seed)
        s.update(model=model, pool=pool, bt=bt, n=c["tokens"], pages=bt.shape[1],
                 image=torch.zeros(bt.shape[1] * model.kv_block_bytes(), dtype=torch.uint8, pin_memory=True))
    return s


def _q(c, seed):
    return _normal((c["batch"], c["n_q_heads"] * c["head_dim"]), 1.0, seed, "q", dtype=torch.float32)


def _ffn(c, seed):
    H, F = c["hidden"], c["ffn"]
    return (_normal((F, H), 0.02, seed, "gate"), _normal((F, H), 0.02, seed, "up"), _normal((H, F), 0.02, seed, "down"),
            _normal((c["rows"], H), 1.0, seed, "x", dtype=torch.float32))


def _linear(c, seed):
    return _normal((c["n"], c["k"]), 0.02, seed, "w"), _normal((c["rows"], c["k"]), 1.0, seed, "x", dtype=torch.float32)


def _prompt(c, seed):
    shape = (c["requests"] * c["tokens"], c["n_kv_heads"], c["head_dim"])
    return _normal(shape, 1.0, seed, "k"), _normal(shape, 1.0, seed, "v")


def run(s):
    kind = s["kind"]
    if kind == "step":
        if s["q_len"] > 1:
            logits = B.decode_step_multi(s["model"], s["pool"], s["bt"], s["lens"], s["tok"], logits=s["logits"])
        else:
            logits = B.decode_step(s["model"], s["pool"], s["bt"], s["lens"], s["tok"], logits=s["logits"])
        return {"logits": logits, "cache": s["cache"]}
    if kind == "attention":
        return B.op_paged_attention(s["model"], s["pool"], 0, s["q"], s["bt"], s["lens"])
    if kind == "ffn":
        return s["gate_up"].ffn(s["down"], s["x"])
    if kind == "linear":
        return s["w"](s["x"])
    if kind == "prefill":
        s["pool"].append(0, s["k"], s["v"], s["bt"], s["seq"], s["pos"])
        return [s["pool"].gather(0, row, s["n"]) for row in s["bt"]]
    s["pool"].swap_out(s["bt"][0], s["pages"], s["image"])
    s["pool"].swap_in(s["bt"][1], s["pages"], s["image"])
    return {"image": s["image"], "restored": s["pool"].gather(0, s["bt"][1], s["n"])}


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def work(c):
    kind = c["kind"]
    if kind == "step":
        rows, H, d = c["batch"] * c["q_len"], c["hidden"], c["head_dim"]
        qn, kn = c["n_q_heads"] * d, c["n_kv_heads"] * d
        params = c["layers"] * (H * (qn + 2 * kn) + qn * H + 3 * H * c["ffn"]) + c["vocab"] * H
        kept = c["batch"] * (_mean_context(c) + c["q_len"])  # cached and new tokens, read once per request
        return {"bytes": 2.0 * params + c["layers"] * 4.0 * kn * (kept + rows) + 4.0 * rows * c["vocab"] + 2.0 * rows * H,
                "flops": 2.0 * rows * params + 4.0 * qn * c["layers"] * c["q_len"] * kept}
    if kind == "attention":
        kept, qn = c["batch"] * _mean_context(c), c["n_q_heads"] * c["head_dim"]
        return {"bytes": 4.0 * c["n_kv_heads"] * c["head_dim"] * kept + 8.0 * c["batch"] * qn, "flops": 4.0 * qn * kept}
    if kind == "ffn":
        return {"bytes": 6.0 * c["hidden"] * c["ffn"] + 8.0 * c["rows"] * c["hidden"], "flops": 6.0 * c["rows"] * c["hidden"] * c["ffn"]}
    if kind == "linear":
        return {"bytes": 2.0 * c["n"] * c["k"] + 4.0 * c["rows"] * (c["n"] + c["k"]), "flops": 2.0 * c["rows"] * c["n"] * c["k"]}
    token = 4.0 * c["n_kv_heads"] * c["head_dim"]
    if kind == "prefill":  # read, written, read, written
        return {"bytes": 4 * token * c["requests"] * c["tokens"], "flops": 0}
    pages = (c["tokens"] + PAGE) // PAGE  # with the next token's
    return {"bytes": 4 * token * PAGE * pages * c["layers"], "flops": 0}


def tolerance(c):
    if c["kind"] in ("prefill", "swap"):
        return "exact"  # pure copies
    if c["kind"] == "step":
        # two bf16 terms per activation and sums in 32 bits: 2e-5 .. 5e-5 from the result in 64 bits; single values of the
        # new K and V may land on the other bf16 neighbour, 2^-8 of themselves
        return {"rel": 2e-4, "max": 1e-2}
    return {"rel": 2e-5, "max": 5e-4}  # 2e-6 .. 5e-6 from the result in 64 bits


# ---- the same in 64 bits -----------------------------------------------------------------------------------------

def _mm(x, w):
    return x @ w.double().t()


def _rms(h, gain):
    return h / torch.sqrt(h.square().mean(-1, keepdim=True) + 1e-5) * gain.double()


def _rope(x, pos, base):
    half = x.shape[-1] // 2
    freq = torch.pow(torch.tensor(float(base), dtype=torch.float64, device=x.device), -torch.arange(half, dtype=torch.float64, device=x.device) / half)
    ang = (pos.double()[..., None] * freq)[..., None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat((a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()), -1)


def _attend(q, k, v, offset):
    """q [t, n_q, d]; k, v [n, n_kv, d]; token j sees the first offset + j positions"""
    t, n_q, d = q.shape
    n, n_kv, _ = k.shape
    q = q.view(t, n_kv, n_q // n_kv, d).permute(1, 0, 2, 3).reshape(n_kv, -1, d)
    s = q @ k.double().permute(1, 2, 0).contiguous() / math.sqrt(d)
    if t > 1:
        seen = torch.arange(n, device=q.device)[None] < (offset + torch.arange(t, device=q.device))[:, None]
        s = s.masked_fill(~seen.repeat_interleave(n_q // n_kv, 0)[None], -math.inf)
    o = torch.softmax(s, -1) @ v.double().permute(1, 0, 2).contiguous()
    return o.view(n_kv, t, n_q // n_kv, d).permute(1, 0, 2, 3).reshape(t, n_q * d)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "linear":
        w, x = _linear(c, seed)
        return _mm(x.double(), w)
    if kind == "ffn":
        wg, wu, wd, x = _ffn(c, seed)
        x = x.double()
        return _mm(torch.nn.functional.silu(_mm(x, wg)) * _mm(x, wu), wd)
    if kind == "prefill":
        k, v = _prompt(c, seed)
        return [(a.double(), b.double()) for a, b in zip(k.split(c["tokens"]), v.split(c["tokens"]))]
    if kind == "swap":
        k, v = _cache(c, c["tokens"], seed, 0, 0)
        return {"image": None, "restored": (k.double(), v.double())}
    lens = _context(c, seed) if kind == "step" else np.maximum(_context(c, seed), 1)
    total, ends = int(lens.sum()), np.cumsum(lens.astype(np.int64))

    def cached(l):
        parts = [_cache(c, total, seed, l, at) for at in range(0, total, CHUNK)]
        empty = [torch.empty((0, c["n_kv_heads"], c["head_dim"]), dtype=torch.bfloat16, device="cuda")]
        return torch.cat([p[0] for p in parts] or empty), torch.cat([p[1] for p in parts] or empty)

    if kind == "attention":
        K, V = cached(0)
        q = _q(c, seed).double().view(c["batch"], 1, c["n_q_heads"], c["head_dim"])
        return torch.cat([_attend(q[i], K[e - n:e], V[e - n:e], n) for i, (n, e) in enumerate(zip(lens.tolist(), ends.tolist()))])
    d, t = c["head_dim"], c["q_len"]
    if c["batch"] * t * c["layers"] < 128:
        # With few rows a handful of new K and V values decides the error: those that lie so close to the middle of two
        # bf16 neighbours that any 32-bit sum may round them either way (about one in two thousand).  Their number, not
        # the precision of the sums, is what a comparison would show.
        return None
    head = _head(c, seed)
    tok = torch.from_numpy(_tokens(c, seed)).cuda().long()
    h = head["embed"][tok].double()  # [batch, t, hidden]
    pos = torch.from_numpy(lens).cuda()[:, None] + torch.arange(t, device="cuda")
    for l in range(c["layers"]):
        w = _layer(c, seed, l)
        K, V = cached(l)
        x = _rms(h, w["attn_norm"])
        q, k, v = (_mm(x, w[n]).view(c["batch"], t, -1, d) for n in ("wq", "wk", "wv"))
        q = _rope(q, pos, c["rope_base"])
        k, v = _rope(k, pos, c["rope_base"]).to(torch.bfloat16), v.to(torch.bfloat16)  # the cache holds bf16
        a = torch.stack([_attend(q[i], torch.cat((K[e - n:e], k[i])), torch.cat((V[e - n:e], v[i])), n + 1)
                         for i, (n, e) in enumerate(zip(lens.tolist(), ends.tolist()))])
        h = h + _mm(a, w["wo"])
        x = _rms(h, w["ffn_norm"])
        h = h + _mm(torch.nn.functional.silu(_mm(x, w["w_gate"])) * _mm(x, w["w_up"]), w["w_down"])
    logits = _mm(_rms(h, head["final_norm"]), head["lm_head"])
    return {"logits": logits if t > 1 else logits[:, 0], "cache": None}
