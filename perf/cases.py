"""Performance cases of the mixed prefill + decode iteration.

One pass is one call of the iteration, the work a server built on this
library has it do: C prompt rows (of one or several prompts, behind cached
prefixes) beside B single-token decodes over the paged KV cache, through all
layers of the context, from the input rows to the output rows with the new
K/V appended to the pools.  Shapes are this repository's own: the 8B-shaped
layer (d 4096, 32/8 heads of 128, FFN 14336) and the Tiny model (d 256, four
heads of 64, FFN 704).

``listed`` names the cases, ``draw`` gives more of the same ranges,
``prepare`` makes what a program holds before the call, ``run`` is the call,
``work`` what it cannot do without, ``exact`` the same results in float64 by
plain torch, and ``tolerance`` how far another correct bf16 implementation
may be from this one.
"""
import math

import numpy as np
import torch

from paper_2609_07883_amd import api

# n_layers is the case's own
SHAPES = {
    "8b": dict(d=4096, hq=32, hkv=8, hd=128, f=14336, theta=500000.0, max_pos=32768),
    "tiny": dict(d=256, hq=4, hkv=4, hd=64, f=704, theta=10000.0, max_pos=4096),
}
EPS = 1e-5
PREFILL = 1      # sequence ids: prompts PREFILL, PREFILL + 1, ..., decodes DECODE, DECODE + 1, ...
DECODE = 100


def _case(name, shape="8b", layers=1, chunk=0, prefix=0, prompts=1, decodes=0, ctx="none", entry="workspace"):
    """chunk: prompt rows in all; prompts: how many prompts they come from;
    prefix: cached tokens of the first prompt (the others start at 0); ctx:
    distribution of the decodes' cached tokens; entry: the ordinary call, or
    the allocation-free one."""
    return dict(name=name, shape=shape, layers=layers, chunk=chunk, prefix=prefix, prompts=prompts,
                decodes=decodes, ctx=ctx, entry=entry)


def listed():
    return [
        # The smallest call: one 128-token chunk of a 512-token prompt of the
        # Tiny model beside four decodes; launches and latency count.
        _case("tiny_c128_p128_b4", shape="tiny", chunk=128, prefix=128, decodes=4, ctx="u64_256"),
        # One user's decode: a single row through a layer, weight streaming.
        _case("decode_b1", decodes=1, ctx="chat"),
        # A lightly loaded server between prompts, through the entry point
        # for callers that may not allocate.
        _case("decode_b8_static", decodes=8, ctx="chat", entry="static"),
        # Decode-only iterations of a stack: each layer reads the last one's rows.
        _case("stack4_decode_b16", layers=4, decodes=16, ctx="u1024_10240"),
        # A chat server's decode batch with no prompt waiting.
        _case("decode_b64", decodes=64, ctx="chat"),
        # A short ragged chunk, no multiple of anything, beside a few decodes.
        _case("ragged_c77_p50_b5", chunk=77, prefix=50, decodes=5, ctx="chat"),
        # Chat bursts: a small chunk beside a full decode batch.
        _case("chat_c64_p960_b256", chunk=64, prefix=960, decodes=256, ctx="chat"),
        # The chunk a tight token deadline leaves, in mid prompt.
        _case("sweep_c256_p2048_b32", chunk=256, prefix=2048, decodes=32, ctx="u512_2048"),
        # Several short prompts taken up in one iteration.
        _case("batched4_c700_b16", chunk=700, prefix=300, prompts=4, decodes=16, ctx="chat"),
        # An ordinary chunk at a prompt's start.
        _case("sweep_c1024_p0_b32", chunk=1024, prefix=0, decodes=32, ctx="u512_2048"),
        # A large chunk of a long prompt.
        _case("sweep_c2048_p8192_b32", chunk=2048, prefix=8192, decodes=32, ctx="u512_2048"),
        # The largest: the last chunk of a 32 K prompt beside long decodes.
        _case("long_c4096_p28672_b8", chunk=4096, prefix=28672, decodes=8, ctx="u16384_32768"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["tiny", "decode", "decode", "stack", "chat", "sweep", "sweep", "batched", "long"])
    if kind == "tiny":
        b = rng.randint(0, 8)
        c = _log_int(rng, 1, 512)
        c = _case("", shape="tiny", layers=rng.randint(1, 3), chunk=c, prefix=rng.randint(0, 512), decodes=b,
                  ctx="u64_256", entry=rng.choice(["workspace", "static"]))
    elif kind == "decode":
        b = _log_int(rng, 1, 256)
        c = _case("", decodes=b, ctx=rng.choice(["chat", "u512_2048", "u1024_10240"]),
                  entry=rng.choice(["workspace", "static"]) if b <= 32 else "workspace")
    elif kind == "stack":
        c = _case("", layers=rng.randint(2, 4), chunk=rng.choice([0, _log_int(rng, 1, 512)]), prefix=rng.randint(0, 4096),
                  decodes=_log_int(rng, 1, 64), ctx="chat")
    elif kind == "chat":
        c = _case("", chunk=_log_int(rng, 8, 512), prefix=rng.randint(0, 4096), decodes=rng.randint(64, 256), ctx="chat")
    elif kind == "sweep":
        c = _case("", chunk=_log_int(rng, 48, 2048), prefix=rng.choice([0, _log_int(rng, 16, 8192)]),
                  decodes=rng.randint(0, 32), ctx="u512_2048")
    elif kind == "batched":
        c = _case("", chunk=_log_int(rng, 64, 2048), prefix=rng.randint(0, 2048), prompts=rng.randint(2, 8),
                  decodes=rng.randint(0, 64), ctx="chat")
    else:
        c = _case("", chunk=_log_int(rng, 512, 4096), prefix=rng.randint(4096, 28672), decodes=rng.randint(4, 8),
                  ctx="u16384_32768")
    del c["name"]
    return c


def _contexts(case):
    """Cached tokens of each decode: fixed by the case."""
    n = case["decodes"]
    rng = np.random.default_rng([2, n])
    if n == 0:
        return []
    if case["ctx"] == "chat":  # log-normal, median 700, sigma 0.8, cap 8192
        v = np.clip(np.rint(700 * np.exp(0.8 * rng.standard_normal(n))), 1, 8192)
    else:
        lo, hi = (int(s) for s in case["ctx"][1:].split("_"))
        v = rng.integers(lo, hi + 1, size=n)
    return [min(int(x), SHAPES[case["shape"]]["max_pos"] - 1) for x in v]


def _prompts(case):
    """(prefix, chunk) of each prompt: the rows split unevenly, the first
    prompt behind its cached prefix and the others at their start."""
    c, n = case["chunk"], min(case["prompts"], case["chunk"])
    if n <= 1:
        return [(case["prefix"], c)] if c else []
    share = np.random.default_rng([7, c, n]).uniform(0.5, 1.5, size=n)
    cut = [0] + [int(x) for x in np.rint(np.cumsum(share) / share.sum() * c)]
    for i in range(1, n + 1):  # every prompt has a row
        cut[i] = min(max(cut[i], cut[i - 1] + 1), c - (n - i))
    return [(case["prefix"] if i == 0 else 0, cut[i + 1] - cut[i]) for i in range(n)]


def _sequences(case):
    """[(id, first new position, new rows)] in row order: prompts, then decodes."""
    seqs = [(PREFILL + i, p, c) for i, (p, c) in enumerate(_prompts(case))]
    return seqs + [(DECODE + i, n, 1) for i, n in enumerate(_contexts(case))]


def _reservations(seqs):
    """The reservations (id, positions) that grow all sequences together, one
    16-token block at a time: pages of a sequence are scattered through the
    pool, as a server leaves them."""
    todo = {sid: at + new for sid, at, new in seqs}
    k = 1
    while todo:
        for sid in list(todo):
            yield sid, min(todo[sid], 16 * k)
            if 16 * k >= todo[sid]:
                del todo[sid]
        k += 1


def _tables(seqs):
    """Block table of each sequence: a reservation takes the lowest free block."""
    tables = {sid: [] for sid, _, _ in seqs}
    for blk, (sid, _) in enumerate(_reservations(seqs)):
        tables[sid].append(blk)
    return tables


def _inputs(case, seed):
    """Weights N(0, 0.02), gains 1 + N(0, 0.02), cached K/V and input rows
    N(0, 1), all bf16, made on the GPU from the seed."""
    s = SHAPES[case["shape"]]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape, std=1.0, mean=0.0):
        t = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        return t.normal_(mean, std, generator=gen)

    qkv = (s["hq"] + 2 * s["hkv"]) * s["hd"]
    weights = [dict(wqkv=normal(qkv, s["d"], std=0.02), wo=normal(s["d"], s["hq"] * s["hd"], std=0.02),
                    wgu=normal(2 * s["f"], s["d"], std=0.02), wd=normal(s["d"], s["f"], std=0.02),
                    g1=normal(s["d"], std=0.02, mean=1.0), g2=normal(s["d"], std=0.02, mean=1.0))
               for _ in range(case["layers"])]
    seqs = _sequences(case)
    blocks = sum(-(-(at + new) // 16) for _, at, new in seqs)
    k_pool = normal(case["layers"], blocks, s["hkv"], s["hd"] // 32, 16, 32)
    v_pool = normal(case["layers"], blocks, s["hkv"], s["hd"], 16)
    x = normal(case["chunk"] + case["decodes"], s["d"])
    return s, weights, k_pool, v_pool, x, seqs, blocks


def prepare(case, seed):
    s, weights, k_pool, v_pool, x, seqs, blocks = _inputs(case, seed)
    ctx = api.Context(case["layers"], s["d"], s["hq"], s["hkv"], s["hd"], s["f"], EPS, s["theta"], s["max_pos"])
    for layer, w in enumerate(weights):
        ctx.set_layer_weights(layer, *(w[k].data_ptr() for k in ("wqkv", "wo", "wgu", "wd", "g1", "g2")))
    ctx.kv_init(k_pool.data_ptr(), v_pool.data_ptr(), blocks)
    for sid, _, _ in seqs:
        ctx.seq_create(sid)
    for sid, n in _reservations(seqs):
        ctx.seq_reserve(sid, n)
    prefills = [q for q in seqs if q[0] < DECODE]
    decodes = [q for q in seqs if q[0] >= DECODE]
    batch = api.Batch.batched(prefills, [q[0] for q in decodes], [q[1] for q in decodes])
    state = dict(ctx=ctx, batch=batch, weights=weights, x=x, y=torch.empty_like(x), k=k_pool, v=v_pool,
                 stream=torch.cuda.current_stream().cuda_stream, static=case["entry"] == "static")
    if not state["static"]:
        n = ctx.workspace_size(case["chunk"], case["decodes"])
        state["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    return state


def run(state):
    ctx, x, y = state["ctx"], state["x"], state["y"]
    if state["static"]:
        ctx.mixed_iteration_static(state["batch"], x.data_ptr(), y.data_ptr(), state["stream"])
    else:
        ws = state["ws"]
        ctx.mixed_iteration(state["batch"], x.data_ptr(), y.data_ptr(), ws.data_ptr(), ws.numel(), state["stream"])
    return {"rows": y, "k": state["k"], "v": state["v"]}


def work(case):
    """Weights, the cached K/V that is attended to, the input rows and the
    new K/V read or written once; the projections' and attention's products."""
    s, n = SHAPES[case["shape"]], case["layers"]
    m = case["chunk"] + case["decodes"]
    qkv = (s["hq"] + 2 * s["hkv"]) * s["hd"]
    params = s["d"] * (qkv + s["hq"] * s["hd"] + 3 * s["f"])
    kv_row = 2 * s["hkv"] * s["hd"] * 2
    cached = sum(at for _, at, _ in _sequences(case))
    pairs = sum(c * at + c * (c + 1) // 2 for _, at, c in _sequences(case))
    return {"bytes": n * (2 * (params + 2 * s["d"]) + kv_row * (cached + m)) + 2 * 2 * m * s["d"],
            "flops": n * (2 * m * params + 4 * s["hq"] * s["hd"] * pairs)}


def tolerance(case):
    """Rows and products' inputs are stored in bf16.  Against float64 one layer
    is 0.0017-0.0046 off and four layers 0.007; two correct implementations
    round at different places, so they may be about twice that apart."""
    return {"rel": 0.01 if case["layers"] == 1 else 0.02, "max": 0.1}


def _norm(x, g):
    return x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS) * g.double()


def _gather(pool, table, is_k, n):
    """[Hkv][n][hd] of one layer's pages, float64 of the bf16 values."""
    p = pool[torch.tensor(table, device=pool.device)]
    if is_k:  # [blocks][Hkv][hd/32][16][32]
        p = p.permute(1, 0, 3, 2, 4).reshape(p.shape[1], -1, p.shape[2] * 32)
    else:     # [blocks][Hkv][hd][16]
        p = p.permute(1, 0, 3, 2).reshape(p.shape[1], -1, p.shape[2])
    return p[:, :n].double()


def exact(case, seed):
    """The layers in float64 with plain torch: RMSNorm, QKV, rotate-half RoPE,
    causal grouped-query attention over cached and new keys, output
    projection, RMSNorm and SwiGLU MLP, both with residuals."""
    s, weights, k_pool, v_pool, x, seqs, _ = _inputs(case, seed)
    hq, hkv, hd = s["hq"], s["hkv"], s["hd"]
    group, half = hq // hkv, hd // 2
    tables = _tables(seqs)
    pos = torch.tensor([at + j for _, at, c in seqs for j in range(c)], device="cuda")
    blk = torch.tensor([tables[sid][(at + j) // 16] for sid, at, c in seqs for j in range(c)], device="cuda")
    ang = pos.double()[:, None] * torch.pow(torch.tensor(s["theta"], dtype=torch.float64, device="cuda"),
                                            -torch.arange(half, device="cuda").double() / half)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def rope(t):
        a, b = t[..., :half], t[..., half:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    x = x.double()
    m = x.shape[0]
    k_all, v_all = [], []
    for layer, w in enumerate(weights):
        qkv = (_norm(x, w["g1"]) @ w["wqkv"].double().T).view(m, hq + 2 * hkv, hd)
        q, k, v = rope(qkv[:, :hq]), rope(qkv[:, hq:hq + hkv]), qkv[:, hq + hkv:]
        out = torch.empty((m, hq, hd), dtype=torch.float64, device="cuda")
        row = 0
        for sid, at, c in seqs:
            keys = torch.cat([_gather(k_pool[layer], tables[sid], True, at), k[row:row + c].transpose(0, 1)], 1)
            vals = torch.cat([_gather(v_pool[layer], tables[sid], False, at), v[row:row + c].transpose(0, 1)], 1)
            hidden = None
            if c > 1:
                hidden = torch.arange(at + c, device="cuda")[None] > pos[row:row + c, None]
            for h in range(hq):
                sc = q[row:row + c, h] @ keys[h // group].T / math.sqrt(hd)
                if hidden is not None:
                    sc.masked_fill_(hidden, -math.inf)
                out[row:row + c, h] = torch.softmax(sc, 1) @ vals[h // group]
            row += c
        kp, vp = k_pool[layer].double(), v_pool[layer].double()
        kp[blk, :, :, pos % 16] = k.reshape(m, hkv, hd // 32, 32)
        vp[blk, :, :, pos % 16] = v
        k_all.append(kp)
        v_all.append(vp)
        x = x + out.view(m, hq * hd) @ w["wo"].double().T
        g, u = (_norm(x, w["g2"]) @ w["wgu"].double().T).split(s["f"], 1)
        x = x + (g / (1 + torch.exp(-g)) * u) @ w["wd"].double().T
    return {"rows": x, "k": torch.stack(k_all), "v": torch.stack(v_all)}
