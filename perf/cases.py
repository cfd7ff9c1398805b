"""The work that a program has this library do, one pass of it per case: a layer of decode attention, a
short stack of decode layers (append + attention), a layer of prompt or API-response processing (append of
many tokens + attention), and a request's blocks going out to host memory and back.

Everything goes through the calls of the ``Lamps`` class on the default stream.  Keys, values and queries
are N(0, 1) in the storage type, block tables a random deal of the pool, the sizes a function of the case
alone, the numbers a function of the seed alone.  Expected results are made by plain torch in 64 bits from
the documented tile layout.
"""
import math
import random

import torch

import paper_2410_18248_amd as P

DEV = "cuda:0"


# ---------------------------------------------------------------- the cases
def _case(name, kind, dtype, heads, batch, ctx, new=(0, 0), spread="log", layers=1, block=16, running=1.0):
    c = {} if name is None else {"name": name}
    c.update(kind=kind, dtype=dtype, H=heads[0], Hkv=heads[1], D=heads[2], block=block, layers=layers, batch=batch,
             ctx_lo=ctx[0], ctx_hi=ctx[1], new_lo=new[0], new_hi=new[1], spread=spread, running=running)
    return c


def listed():
    return [
        # one user, one layer of an 8B model with grouped heads: the latency of the smallest decode call
        _case("decode_one_request", "decode", "bf16", (32, 8, 128), 1, (1999, 1999)),
        # the serving loop's decode iteration: append + attention for each of 4 layers of a 13B model
        _case("serving_step", "step", "bf16", (40, 40, 128), 16, (60, 1500), layers=4),
        # a 7B model's batch, a fifth of it waiting for API calls
        _case("decode_7b", "decode", "bf16", (32, 32, 128), 64, (128, 2048), spread="even", running=0.8),
        # a large batch of an 8B model with grouped heads, contexts from a line to a document
        _case("decode_8b_gqa", "decode", "bf16", (32, 8, 128), 256, (32, 8192), running=0.9),
        # long documents in blocks of 32
        _case("decode_long_gqa", "decode", "bf16", (32, 8, 128), 32, (4096, 32768), spread="even", block=32, running=0.6),
        # 32-bit storage, as a program that checks its model's numbers has it
        _case("decode_f32", "decode", "f32", (32, 8, 128), 24, (17, 2500)),
        # long prompts (or discarded contexts) of an 8B model, nothing cached before
        _case("prompt_gqa", "prompt", "bf16", (32, 8, 128), 4, (0, 0), (4096, 4096)),
        # an iteration's new requests on a 13B model: ragged prompts of a few words to a page
        _case("prompts_13b", "prompt", "bf16", (40, 40, 128), 24, (0, 0), (16, 700)),
        # API responses: a few tokens each, processed over what the requests kept in the cache
        _case("api_responses", "prompt", "bf16", (32, 8, 128), 12, (300, 3000), (4, 64)),
        # a chunk of a recompute on a 6B model with head size 256
        _case("chunk_d256", "prompt", "bf16", (16, 16, 256), 4, (512, 2048), (512, 512)),
        # prompts in 32-bit storage
        _case("prompt_f32", "prompt", "f32", (8, 8, 64), 6, (0, 0), (17, 700)),
        # a request enters an API call and returns: 48 blocks of 32 layers out to pinned memory and back
        _case("swap_out_in", "swap", "bf16", (32, 8, 128), 1, (768, 768), layers=32),
    ]


HEADS = [(32, 32, 128), (32, 8, 128), (40, 40, 128), (16, 16, 256), (8, 2, 64), (32, 4, 128), (8, 8, 64)]
HEADS_F32 = [(8, 8, 64), (32, 8, 128), (8, 2, 32), (32, 32, 64)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "step", "prompt", "prompt", "prompt", "swap"])
    if kind == "swap":
        return _case(None, "swap", "bf16", rng.choice([(32, 8, 128), (32, 32, 128)]), 1, (n := _log(rng, 16, 700), n),
                     layers=rng.choice([1, 8, 16, 32]))
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    heads = rng.choice(HEADS_F32 if dtype == "f32" else HEADS)
    token = 2 * heads[1] * heads[2] * (4 if dtype == "f32" else 2)   # bytes of one cached position
    block = rng.choice([16, 16, 16, 32])
    if kind == "step":
        batch = _log(rng, 1, 32)
        return _case(None, kind, dtype, heads, batch, (_log(rng, 16, 64), _log(rng, 100, 1500)), layers=rng.choice([2, 4]), block=block)
    if kind == "decode":
        batch = _log(rng, 1, 256)
        most = max(64, min(32768, int(1.5e9 / token / batch)))
        lo = _log(rng, 16, most)
        return _case(None, kind, dtype, heads, batch, (lo, _log(rng, lo, most)), spread=rng.choice(["log", "even"]), block=block,
                     running=rng.choice([1.0, 0.9, 0.6]))
    if rng.random() < 0.5:                                            # prompts: nothing cached
        batch = _log(rng, 1, 32)
        most = max(32, min(4096, (2000 if dtype == "f32" else 16000) // batch))
        lo = _log(rng, 8, most)
        return _case(None, kind, dtype, heads, batch, (0, 0), (lo, _log(rng, lo, most)), block=block)
    batch = _log(rng, 1, 32)                                          # API responses and chunks of a recompute
    hi = _log(rng, 2, max(4, min(512, (500 if dtype == "f32" else 4000) // batch)))
    lo = _log(rng, 64, 1000)
    return _case(None, kind, dtype, heads, batch, (lo, _log(rng, lo, 4000)), (max(1, hi // 4), hi), block=block)


# ---------------------------------------------------------------- sizes
def _sizes(c):
    """(cached tokens, new tokens, running) per request: a function of the case alone."""
    rng = random.Random("%(ctx_lo)d %(ctx_hi)d %(new_lo)d %(new_hi)d %(batch)d %(H)d %(Hkv)d" % c)

    def pick(lo, hi):
        return rng.randint(lo, hi) if c["spread"] == "even" or lo < 1 else min(hi, max(lo, _log(rng, lo, hi)))

    B = c["batch"]
    ctx = [pick(c["ctx_lo"], c["ctx_hi"]) for _ in range(B)]
    new = [pick(c["new_lo"], c["new_hi"]) for _ in range(B)]
    away = set(rng.sample(range(B), int(round((1.0 - c["running"]) * B))))
    return ctx, new, [0 if r in away and len(away) < B else 1 for r in range(B)]


def _blocks(c):
    ctx, new, _ = _sizes(c)
    grow = 1 if c["kind"] == "step" else 0
    return [(a + b + grow + c["block"] - 1) // c["block"] for a, b in zip(ctx, new)]


def work(c):
    ctx, new, run = _sizes(c)
    es = 4 if c["dtype"] == "f32" else 2
    token, row = 2 * c["Hkv"] * c["D"] * es, c["H"] * c["D"] * es
    if c["kind"] == "swap":                                  # each block is read and written once each way
        return {"bytes": 4 * sum(_blocks(c)) * c["layers"] * token * c["block"], "flops": 0}
    if c["kind"] == "prompt":
        pairs = sum(b * a + b * (b + 1) // 2 for a, b in zip(ctx, new))
        return {"bytes": sum(a * token + b * (2 * token + 2 * row) for a, b in zip(ctx, new)), "flops": 4 * c["D"] * c["H"] * pairs}
    grow = 1 if c["kind"] == "step" else 0
    seen = sum(a + grow for a, on in zip(ctx, run) if on)
    n = sum(run)
    return {"bytes": c["layers"] * (seen * token + n * (2 * row + grow * token)),
            "flops": c["layers"] * 4 * c["D"] * c["H"] * seen}


def tolerance(c):
    if c["kind"] == "swap":
        return "exact"
    # measured against 64 bits: bf16 1.6e-3 to 2.3e-3 (its output's rounding), 32 bits 1.1e-7 to 1.5e-7
    # (more terms in a chain, up to 32 000 positions in one, cost a few times that)
    return {"rel": 8e-3} if c["dtype"] == "bf16" else {"rel": 1e-6}


# ---------------------------------------------------------------- inputs
def _type(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _inputs(c, seed):
    """What the call is given, as tensors on the GPU."""
    g = torch.Generator(DEV).manual_seed(seed)
    ctx, new, run = _sizes(c)
    nblk = _blocks(c)
    B, L, D, bs = c["batch"], c["layers"], c["D"], c["block"]
    spare = sum(nblk) if c["kind"] == "swap" else 0          # the swap comes back to other blocks
    pool_blocks = sum(nblk) + spare + sum(nblk) // 10 + 1

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=_type(c))

    s = {"k_pool": normal(pool_blocks, L, c["Hkv"], bs * D), "v_pool": normal(pool_blocks, L, c["Hkv"], bs * D)}
    order = torch.randperm(pool_blocks, generator=g, device=DEV).tolist()
    table, at = torch.full((B, max(nblk)), -1, dtype=torch.int32), 0
    for r, n in enumerate(nblk):
        table[r, :n] = torch.tensor(order[at:at + n], dtype=torch.int32)
        at += n
    s["ids"], s["back"] = order[:sum(nblk)], order[sum(nblk):sum(nblk) + spare]
    s["table"] = table.to(DEV)
    s["ctx"] = torch.tensor([a + b for a, b in zip(ctx, new)], dtype=torch.int32, device=DEV)
    s["mask"] = torch.tensor(run, dtype=torch.uint8, device=DEV)
    rows = sum(new) if c["kind"] == "prompt" else B
    lead = (L,) if c["kind"] == "step" else ()
    if c["kind"] != "swap":
        s["q"] = normal(*lead, rows, c["H"], D)
        s["k_new"] = normal(*lead, rows, c["Hkv"], D)
        s["v_new"] = normal(*lead, rows, c["Hkv"], D)
        s["out"] = torch.zeros_like(s["q"])
    start = [0]
    for n in new:
        start.append(start[-1] + n)
    s["q_start"] = torch.tensor(start, dtype=torch.int32, device=DEV)
    s["total"], s["max_new"] = start[-1], max(new)
    return s


class _State:
    """Pools, workspace, context and arguments, as a serving program keeps them."""

    def __init__(self, c, seed):
        self.case, self.lam = c, None
        self.__dict__.update(_inputs(c, seed))
        cfg = P.LampsConfig(c["layers"], c["H"], c["Hkv"], c["D"], c["block"], self.k_pool.shape[0], self.table.shape[1],
                            c["batch"], P.LAMPS_F32 if c["dtype"] == "f32" else P.LAMPS_BF16)
        self.ws = torch.empty(P.lamps_workspace_bytes(cfg), dtype=torch.uint8, device=DEV)
        self.so, self.si = torch.cuda.Stream(DEV), torch.cuda.Stream(DEV)
        self.lam = P.Lamps(cfg, self.k_pool, self.v_pool, self.ws, 0, self.so.cuda_stream, self.si.cuda_stream)
        self.lam.alloc_blocks(self.k_pool.shape[0])
        self.grown = self.ctx + 1
        if c["kind"] == "swap":
            self.host = torch.zeros(len(self.ids) * P.lamps_block_bytes(cfg), dtype=torch.uint8, pin_memory=True)

    def __del__(self):
        if self.lam is not None:
            self.lam.destroy()


def prepare(c, seed):
    return _State(c, seed)


def run(s):
    c, lam = s.case, s.lam
    if c["kind"] == "decode":
        lam.decode_attn(0, c["batch"], s.q, s.table, s.ctx, s.mask, s.out)
        return s.out
    if c["kind"] == "step":
        for layer in range(c["layers"]):
            lam.kv_append(layer, c["batch"], s.k_new[layer], s.v_new[layer], s.table, s.ctx, s.mask, False)
            lam.decode_attn(layer, c["batch"], s.q[layer], s.table, s.grown, s.mask, s.out[layer])
        return [s.out, s.k_pool, s.v_pool]
    if c["kind"] == "prompt":
        lam.kv_append_tokens(0, c["batch"], s.total, s.k_new, s.v_new, s.q_start, s.table, s.ctx)
        lam.prefill_attn(0, c["batch"], s.total, s.q, s.q_start, s.table, s.ctx, s.out, max_new_tokens=s.max_new)
        return [s.out, s.k_pool, s.v_pool]
    lam.swap_out(s.ids, s.host)                              # the swap-in is ordered behind it by the library
    ticket = lam.swap_in(s.host, s.back)
    lam.ticket_wait(ticket)
    return [s.host, s.k_pool, s.v_pool]


# ---------------------------------------------------------------- expected results
def _logical(c, x, value):
    """Tiles [n][Hkv][block * D] -> [n][Hkv][block][D]."""
    n, D, u = x.shape[0], c["D"], c["block"] // 16
    if c["dtype"] == "f32" or c["H"] == c["Hkv"]:
        return x.view(n, c["Hkv"], c["block"], D)
    if not value:                                            # [sub-tile][d / 8][slot][8]
        x = x.view(n, c["Hkv"], u, D // 8, 16, 8).permute(0, 1, 2, 4, 3, 5)
    else:                                                    # [sub-tile][d / 32][slot / 4][d % 16][d % 32 / 16][slot % 4]
        x = x.view(n, c["Hkv"], u, D // 32, 4, 16, 2, 4).permute(0, 1, 2, 4, 7, 3, 6, 5)
    return x.reshape(n, c["Hkv"], c["block"], D)


def _tiles(c, x, value):
    """The other way."""
    n, D, u = x.shape[0], c["D"], c["block"] // 16
    if c["dtype"] != "f32" and c["H"] != c["Hkv"]:
        if not value:
            x = x.reshape(n, c["Hkv"], u, 16, D // 8, 8).permute(0, 1, 2, 4, 3, 5)
        else:
            x = x.reshape(n, c["Hkv"], u, 4, 4, D // 32, 2, 16).permute(0, 1, 2, 5, 3, 7, 6, 4)
    return x.reshape(n, c["Hkv"], c["block"] * D)


def _attend(c, q, k, v, first):
    """q [n][H][D] at positions first .. first + n - 1 over k, v [Hkv][C][D], in 64 bits."""
    n, G, out = q.shape[0], c["H"] // c["Hkv"], torch.empty(q.shape, dtype=torch.float64, device=q.device)
    seen = torch.arange(k.shape[1], device=q.device)[None, :] <= first + torch.arange(n, device=q.device)[:, None]
    for g in range(c["Hkv"]):
        kt, vd = k[g].double().t().contiguous(), v[g].double()
        for h in range(g * G, (g + 1) * G):
            w = torch.softmax((q[:, h].double() @ kt / math.sqrt(c["D"])).masked_fill_(~seen, -math.inf), 1)
            out[:, h] = w @ vd
    return out


def exact(c, seed):
    s = _inputs(c, seed)
    kp, vp = s["k_pool"], s["v_pool"]
    if c["kind"] == "swap":
        ids, back = torch.tensor(s["ids"], device=DEV), torch.tensor(s["back"], device=DEV)
        images = torch.stack([kp[ids].flatten(1), vp[ids].flatten(1)], 1)
        kp[back], vp[back] = kp[ids], vp[ids]
        return [images.view(torch.uint8).flatten(), kp, vp]
    ctx, new, run = _sizes(c)
    out = torch.zeros(s["q"].shape, dtype=torch.float64, device=DEV)
    for layer in range(c["layers"]):
        q, o = (s["q"][layer], out[layer]) if c["kind"] == "step" else (s["q"], out)
        kn, vn = (s["k_new"][layer], s["v_new"][layer]) if c["kind"] == "step" else (s["k_new"], s["v_new"])
        at = 0
        for r in range(c["batch"]):
            n = new[r] if c["kind"] == "prompt" else 1
            if run[r] and n:
                ids = s["table"][r, :_blocks(c)[r]].long()
                k = _logical(c, kp[ids, layer], False).transpose(0, 1).reshape(c["Hkv"], -1, c["D"])
                v = _logical(c, vp[ids, layer], True).transpose(0, 1).reshape(c["Hkv"], -1, c["D"])
                if c["kind"] != "decode":                    # the new tokens join the cache
                    k, v = k.clone(), v.clone()
                    k[:, ctx[r]:ctx[r] + n] = kn[at:at + n].transpose(0, 1)
                    v[:, ctx[r]:ctx[r] + n] = vn[at:at + n].transpose(0, 1)
                    kp[ids, layer] = _tiles(c, k.view(c["Hkv"], len(ids), c["block"], c["D"]).transpose(0, 1), False)
                    vp[ids, layer] = _tiles(c, v.view(c["Hkv"], len(ids), c["block"], c["D"]).transpose(0, 1), True)
                end = ctx[r] + (n if c["kind"] != "decode" else 0)
                o[at:at + n] = _attend(c, q[at:at + n], k[:, :end], v[:, :end], end - n)
            at += n
    return out if c["kind"] == "decode" else [out, kp, vp]
