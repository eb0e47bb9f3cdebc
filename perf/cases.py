"""Performance cases of kvx: one attention layer of a serving step, as a user runs it.

A case is one layer's work for one batch of requests through the public calls of
``paper_2609_32278_amd.kvx``: the suffix K/V go into the paged pool (``store_kv``,
or ``store_kv_rope`` with the norm and rotation fused) and the suffix queries attend
over cached prefix and suffix (``extend_attention``).  Kinds:

  turn   store, then attention: what every layer does at a turn start or decode step
  store  the store alone (a long recompute hands its K/V over layer by layer)
  pages  whole pages out of one pool and into another (moving a request's KV)

Head shapes are those of the repository's workloads and tests (32/8/128, 64/8/128,
8/2/64, 4/2/64) and one tensor-parallel shard (8/1/128).  Lengths follow from the case
alone (``lens`` seeds them), values and page placement from the seed of ``prepare``.
Page moves to pinned host memory are bound by the host link and are not listed.
"""

import math
import random

import numpy as np
import torch

from paper_2609_32278_amd import kvx

PAGE = 16
THETA, EPS = 1e6, 1e-6  # rotary base and norm epsilon of the Qwen3-shaped fused store

# ------------------------------------------------------------------- the cases


def _turn(name, heads, d, n, p, e, **more):
    """n requests with prefixes in [p0, p1] (log-uniform) and suffixes in [e0, e1], and
    `ones` further requests that decode one token over prefixes of [q0, q1]."""
    c = {"name": name, "kind": "turn", "hq": heads[0], "hkv": heads[1], "d": d, "n": n, "p0": p[0], "p1": p[1],
         "e0": e[0], "e1": e[1], "ones": 0, "q0": 0, "q1": 0, "fp8": False, "rope": True, "scaled_q": False,
         "noalloc": False, "lse": False, "sigma": 1.0, "whole": False, "lens": 1}
    c.update(more)
    return c


def listed():
    llama, wide = (32, 8), (64, 8)
    return [
        # the smallest step: the 4-request correctness batch (head_dim 64); all latency and launches
        _turn("tiny_turn", (4, 2), 64, 4, (16, 512), (8, 100), rope=False),
        # interactive decode: a handful of agents, one token each; launches and a nearly idle chip
        _turn("decode_few", llama, 128, 4, (1000, 8000), (1, 1)),
        # a full decode batch of returning agents (128 agents, 4k-32k contexts)
        _turn("decode_llama8b", llama, 128, 128, (4096, 32768), (1, 1), sigma=0.5),
        # long-context decode on an fp8 pool, 70B-shaped heads
        _turn("decode_fp8_long", wide, 128, 24, (16384, 131072), (1, 1), fp8=True),
        # continuous batching: three turn starts prefill while 61 agents decode in the same step
        _turn("mixed_serving", llama, 128, 3, (4096, 16384), (256, 2048), ones=61, q0=1024, q1=16384),
        # short turns: tool outputs of a few dozen tokens on long cached histories
        _turn("short_turns", llama, 128, 24, (2048, 49152), (8, 160)),
        # the same on small heads (the agent replay's 8/2/64 layer), ragged and unaligned
        _turn("short_turns_d64", (8, 2), 64, 12, (300, 9000), (20, 700), rope=False, lse=True),
        # turn starts of 16 returning agents with partial hits (Llama-3-8B-shaped layer)
        _turn("llama8b", llama, 128, 16, (4096, 32768), (64, 2048), rope=False, sigma=0.5),
        # the headline shape: a 70B-shaped layer with long prefixes and thousands of new tokens
        _turn("wide70b", wide, 128, 12, (16384, 131072), (512, 4096)),
        # the same on an fp8 pool
        _turn("wide70b_fp8", wide, 128, 12, (16384, 131072), (512, 4096), fp8=True, lens=2),
        # one fully evicted agent recomputes its whole context (prefix 0), alone on the GPU;
        # scaled-Q, the option for prefill throughput
        _turn("recompute_scaled_q", llama, 128, 1, (0, 0), (32768, 32768), scaled_q=True),
        # moving 2000 pages (32k tokens) of KV between pools, canonical buffers in between
        {"name": "move_pages", "kind": "pages", "hkv": 8, "d": 128, "n": 2000, "fp8": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: decode, short and long turns, recomputes, mixed
    steps, stores and page moves, over the head shapes, pool types and options above."""
    kind = rng.choice(["decode", "decode", "short", "turn", "turn", "mixed", "recompute", "store", "pages"])
    heads, d = rng.choice([((32, 8), 128), ((32, 8), 128), ((64, 8), 128), ((8, 1), 128), ((8, 2), 64), ((4, 2), 64)])
    lens = rng.randrange(1 << 20)
    if kind == "pages":
        return {"kind": "pages", "hkv": heads[1], "d": d, "n": _log(rng, 7, 4000), "fp8": rng.random() < 0.5}
    more = {"fp8": rng.random() < 0.35, "rope": rng.random() < 0.6, "lse": rng.random() < 0.3, "lens": lens,
            "sigma": rng.choice([0.5, 1.0]), "whole": rng.random() < 0.5}
    while True:
        if kind == "decode":
            a = _log(rng, 300, 40000)
            c = _turn("", heads, d, _log(rng, 1, 160), (a, _log(rng, a, 131072)), (1, 1),
                      noalloc=rng.random() < 0.25, **more)
        elif kind == "short":
            a = _log(rng, 200, 30000)
            e = _log(rng, 2, 200)
            c = _turn("", heads, d, _log(rng, 1, 40), (a, _log(rng, a, 65536)), (e, _log(rng, e, 400)),
                      noalloc=rng.random() < 0.15, **more)
        elif kind == "turn":
            a = _log(rng, 500, 50000)
            e = _log(rng, 64, 3000)
            c = _turn("", heads, d, _log(rng, 1, 40), (a, _log(rng, a, 131072)), (e, _log(rng, e, 8192)),
                      scaled_q=rng.random() < 0.3, **more)
        elif kind == "mixed":
            a, b = _log(rng, 500, 20000), _log(rng, 500, 20000)
            e = _log(rng, 16, 1000)
            c = _turn("", heads, d, _log(rng, 1, 8), (a, 2 * a), (e, 3 * e), ones=_log(rng, 4, 96), q0=b, q1=2 * b,
                      **more)
        elif kind == "recompute":
            e = _log(rng, 1000, 32768)
            c = _turn("", heads, d, rng.choice([1, 1, 2, 3]), (0, 0), (e, e), scaled_q=rng.random() < 0.3, **more)
        else:
            c = _turn("", heads, d, _log(rng, 1, 60), (0, 4096), (64, 8192), **more)
            c["kind"] = "store"
        del c["name"]
        w = work(c)
        if w["flops"] <= 4e13 and w["bytes"] <= 6e9:
            return c


# ------------------------------------------------------------------ one case's batch


def _lengths(c):
    """(prefix, suffix) token counts of the case's requests; `whole` prefixes end on a page."""
    rng = random.Random(c["lens"])
    p, e = [], []
    for i in range(c["n"] + c["ones"]):
        lo, hi = (c["p0"], c["p1"]) if i < c["n"] else (c["q0"], c["q1"])
        x = int(math.exp(rng.uniform(math.log(lo + 1), math.log(hi + 1)))) - 1 if hi > lo else lo
        p.append(x // PAGE * PAGE if c["whole"] else x)
        e.append(rng.randint(c["e0"], c["e1"]) if i < c["n"] else 1)
    both = list(zip(p, e))
    rng.shuffle(both)  # decoding and prefilling requests share the batch in no order
    return np.array([x[0] for x in both], np.int64), np.array([x[1] for x in both], np.int64)


def work(case):
    """What one pass cannot do without: Q, K and V of the suffix read, Q (rotated) and K/V
    written, each cached K/V row and each output row once; 4 d flop per visible (row, key)."""
    hkv, d = case["hkv"], case["d"]
    eb = 1 if case["fp8"] else 2
    if case["kind"] == "pages":
        return {"bytes": 8 * case["n"] * hkv * PAGE * d * eb, "flops": 0}
    p, e = _lengths(case)
    t, hq = int(e.sum()), case["hq"]
    store = 2 * t * hkv * d * (2 + eb) + (4 * t * hq * d if case["rope"] else 0)
    if case["kind"] == "store":
        return {"bytes": store, "flops": 0}
    attn = 4 * t * hq * d + 2 * int((p + e).sum()) * hkv * d * eb + (4 * t * hq if case["lse"] else 0)
    return {"bytes": store + attn, "flops": 4 * d * hq * int((e * p + e * (e + 1) // 2).sum())}


class _Owner:
    """Owns a pool handle; the pool is freed when the last view of its memory is gone."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        kvx.kv_pool_destroy(self.handle)


class _Memory:
    """`n` elements of the pool's memory, for torch.as_tensor, which keeps this object (and so
    the pool) alive as long as the tensor's storage."""

    def __init__(self, owner, base, n, typestr):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": typestr, "data": (base, False), "version": 3}


class _Pool:
    """A KV pool and its memory as tensors [page][kv_head][slot][dim]."""

    def __init__(self, pages, hkv, d, fp8, scales):
        dtype = kvx.KVX_KV_FP8_E4M3 if fp8 else kvx.KVX_KV_BF16
        self.handle = kvx.kv_pool_create(pages, PAGE, hkv, d, dtype, *scales)
        owner = _Owner(self.handle)
        lay = kvx.kv_pool_layout(self.handle)
        shape = (pages, hkv, PAGE, d)

        def view(x):
            flat = torch.as_tensor(_Memory(owner, lay[x + "_base"], math.prod(shape), "|u1" if fp8 else "<i2"),
                                   device="cuda")
            strides = [lay[f"{x}_stride_{a}"] for a in ("page", "head", "slot", "dim")]
            return (flat if fp8 else flat.view(torch.bfloat16)).as_strided(shape, strides)

        self.owner, self.k, self.v = owner, view("k"), view("v")


def _randn(gen, shape, sigma=1.0):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(sigma)


def _inputs(c, seed):
    """The case's tensors and page tables, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng([31, seed])
    hkv, d = c["hkv"], c["d"]
    s = {"scales": (None, None)}
    if c["fp8"]:
        s["scales"] = tuple(rng.uniform(0.01, 0.1, hkv).astype(np.float32) for _ in range(2))
    if c["kind"] == "pages":
        s["pages"] = int(1.5 * c["n"]) + 1
        s["from"], s["to"] = [rng.permutation(s["pages"])[:c["n"]].astype(np.int32) for _ in range(2)]
        shape = (s["pages"], hkv, PAGE, d)
        if c["fp8"]:  # any code but the NaN ones
            s["k"], s["v"] = [torch.randint(0, 127, shape, generator=gen, device="cuda", dtype=torch.uint8)
                              for _ in range(2)]
        else:
            s["k"], s["v"] = _randn(gen, shape), _randn(gen, shape)
        return s
    p, e = _lengths(c)
    need = -(-(p + e) // PAGE)
    s["pages"] = int(need.sum() * 1.1) + 8
    s["indptr"] = np.concatenate([[0], np.cumsum(need)]).astype(np.int32)
    s["ids"] = rng.permutation(s["pages"])[:int(need.sum())].astype(np.int32)
    s["p"], s["e"] = p, e
    t, h, sg = int(e.sum()), int(p.sum()), c["sigma"]
    s["q"] = _randn(gen, (t, c["hq"], d), sg)
    s["k_ext"], s["v_ext"] = _randn(gen, (t, hkv, d), sg), _randn(gen, (t, hkv, d), sg)
    s["k_hist"], s["v_hist"] = _randn(gen, (h, hkv, d), sg), _randn(gen, (h, hkv, d), sg)
    s["q_norm"], s["k_norm"] = [(torch.rand(d, generator=gen, device="cuda") + 0.5).to(torch.bfloat16)
                                for _ in range(2)]
    return s


def _table(ids):
    return torch.from_numpy(ids).cuda()


def prepare(case, seed):
    """What a serving program holds before the call: the pool with the cached prefixes, the
    batch with its page table, the layer's Q, K and V, and output buffers."""
    c, s = case, _inputs(case, seed)
    s["case"] = c
    if c["kind"] == "pages":
        s["src"] = _Pool(s["pages"], c["hkv"], c["d"], c["fp8"], s["scales"])
        s["dst"] = _Pool(s["pages"], c["hkv"], c["d"], c["fp8"], s["scales"])
        s["src"].k.copy_(s["k"])
        s["src"].v.copy_(s["v"])
        s["k_lin"], s["v_lin"] = [torch.empty(c["n"], *s["k"].shape[1:], dtype=s["k"].dtype, device="cuda")
                                  for _ in range(2)]
        del s["k"], s["v"]
        return s
    s["pool"] = _Pool(s["pages"], c["hkv"], c["d"], c["fp8"], s["scales"])
    kvx.kv_pool_set_scaled_q(s["pool"].handle, c["scaled_q"])
    if s["k_hist"].numel():  # an earlier turn wrote the prefixes
        need = -(-s["p"] // PAGE)
        ids = np.concatenate([s["ids"][a:a + n] for a, n in zip(s["indptr"], need)])
        past = kvx.Batch(np.zeros_like(s["p"]), s["p"], np.concatenate([[0], np.cumsum(need)]), _table(ids))
        kvx.store_kv(s["pool"].handle, past, s["k_hist"], s["v_hist"])
    torch.cuda.synchronize()
    del s["k_hist"], s["v_hist"]
    s["batch"] = kvx.Batch(s["p"], s["e"], s["indptr"], _table(s["ids"]))
    s["q_rot"] = torch.empty_like(s["q"]) if c["rope"] else s["q"]
    s["out"] = torch.empty_like(s["q"])
    s["lse"] = torch.empty(s["q"].shape[:2], dtype=torch.float32, device="cuda") if c["lse"] else None
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "pages":
        kvx.kv_pool_read_pages(s["src"].handle, s["from"], s["k_lin"], s["v_lin"])
        kvx.kv_pool_write_pages(s["dst"].handle, s["to"], s["k_lin"], s["v_lin"])
        return {"k_lin": s["k_lin"], "v_lin": s["v_lin"], "k": s["dst"].k, "v": s["dst"].v}
    pool, batch = s["pool"].handle, s["batch"]
    got = {"k": s["pool"].k, "v": s["pool"].v}
    if c["rope"]:
        kvx.store_kv_rope(pool, batch, s["k_ext"], s["v_ext"], theta=THETA, rotary_dim=c["d"], q=s["q"],
                          num_q_heads=c["hq"], q_out=s["q_rot"], q_norm=s["q_norm"], k_norm=s["k_norm"], norm_eps=EPS)
        got["q_rot"] = s["q_rot"]
    else:
        kvx.store_kv(pool, batch, s["k_ext"], s["v_ext"])
    if c["kind"] == "turn":
        attend = kvx.extend_attention_noalloc if c["noalloc"] else kvx.extend_attention
        attend(pool, batch, s["q_rot"], c["hq"], c["d"] ** -0.5, s["out"], s["lse"])
        got["out"] = s["out"]
        if c["lse"]:
            got["lse"] = s["lse"]
    return got


def tolerance(case):
    """Copies and page moves are exact.  The rotation is float32 rounded once: values at a
    rounding boundary may differ by one bf16 step (2^-8), fp8 codes by one code, and few do.
    Attention rounds P and the output to bf16: 2.3e-3 rms away from exact attention."""
    if case["kind"] == "pages" or (case["kind"] == "store" and not case["rope"]):
        return "exact"
    if case["kind"] == "store":
        return {"rel": 2e-4, "max": 1e-2, "differ": 1e-3}
    return {"rel": 1e-2, "max": 0.05, "differ": 1e-3}


# ------------------------------------------------------------------ in 64 bits


def _rotate(x, w, pos):
    """RMS norm with weight w and half-layout rotary embedding at positions pos, in 64 bits."""
    d = x.shape[-1]
    x = x.double()
    x = x / (x.square().mean(-1, keepdim=True) + float(np.float32(EPS))).sqrt() * w.double()
    rate = THETA ** (-torch.arange(0, d, 2, dtype=torch.float64, device=x.device) / d)
    a = pos.double()[:, None, None] * rate
    lo, hi = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([lo * a.cos() - hi * a.sin(), lo * a.sin() + hi * a.cos()], -1)


def _stored(x, scale):
    """The 64-bit values a pool holds for x: bf16, or e4m3 codes times the head's scale."""
    if scale is None:
        return x.to(torch.bfloat16).double()
    s = torch.from_numpy(scale).cuda()
    inv = (1.0 / s)[:, None]
    code = (x.float() * inv).clamp(-448, 448).to(torch.float8_e4m3fn)
    return code.double() * s.double()[:, None]


def exact(case, seed):
    c = case
    if c["kind"] == "pages" or work(c)["flops"] > 8e13:
        return None
    s = _inputs(c, seed)
    p, e, g = s["p"], s["e"], c["hq"] // c["hkv"]
    where = torch.from_numpy(np.concatenate([np.arange(a, a + n) for a, n in zip(p, e)])).cuda()
    q, k = s["q"].double(), s["k_ext"].double()
    if c["rope"]:
        q, k = _rotate(s["q"], s["q_norm"], where), _rotate(s["k_ext"], s["k_norm"], where)
    got = {"k": None, "v": None}
    if c["rope"]:
        got["q_rot"] = q
    qb = q.to(torch.bfloat16).double()  # attention takes the rounded queries
    ks, vs = s["scales"]
    if not c["fp8"]:  # the whole pool: zero pages, the prefixes, the suffix (K before its rounding)
        got["k"], got["v"] = [torch.zeros(s["pages"], PAGE, c["hkv"], c["d"], device="cuda", dtype=torch.float64)
                              for _ in range(2)]
    out = torch.empty_like(q)
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device="cuda")
    row = past = 0
    for r in range(len(p)):
        pr, er = int(p[r]), int(e[r])
        kh, vh = s["k_hist"][past:past + pr], s["v_hist"][past:past + pr]
        if not c["fp8"]:
            t = np.arange(pr + er)
            page = torch.from_numpy(s["ids"][s["indptr"][r] + t // PAGE].astype(np.int64)).cuda()
            slot = torch.from_numpy(t % PAGE).cuda()
            got["k"][page, slot] = torch.cat([kh.double(), k[row:row + er]])
            got["v"][page, slot] = torch.cat([vh, s["v_ext"][row:row + er]]).double()
        if c["kind"] == "turn":
            kk = torch.cat([_stored(kh, ks), _stored(k[row:row + er], ks)])
            vv = torch.cat([_stored(vh, vs), _stored(s["v_ext"][row:row + er], vs)])
            step = max(1, (1 << 28) // (g * (pr + er)))
            for a in range(0, er, step):
                b = min(er, a + step)
                n = pr + b
                hide = torch.arange(n, device="cuda") > torch.arange(pr + a, pr + b, device="cuda")[:, None]
                for h in range(c["hkv"]):
                    x = qb[row + a:row + b, h * g:(h + 1) * g].reshape(-1, c["d"])
                    x = (x @ kk[:n, h].T).mul_(c["d"] ** -0.5).view(b - a, g, n)
                    x = x.masked_fill_(hide[:, None], -math.inf).view(-1, n)
                    top = x.amax(-1, keepdim=True)
                    x = x.sub_(top).exp_()
                    total = x.sum(-1, keepdim=True)
                    out[row + a:row + b, h * g:(h + 1) * g] = ((x @ vv[:n, h]) / total).view(b - a, g, -1)
                    lse[row + a:row + b, h * g:(h + 1) * g] = (top + total.log()).view(b - a, g)
        row, past = row + er, past + pr
    if not c["fp8"]:
        got["k"], got["v"] = [x.transpose(1, 2) for x in (got["k"], got["v"])]
    if c["kind"] == "turn":
        got["out"] = out
        if c["lse"]:
            got["lse"] = lse
    return got
