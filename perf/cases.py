"""The calls whose speed counts: what a serving or evaluation program that keeps a pruned KV cache has
librap do, over the sizes, widths and cache kinds that this repository's workloads, tests and benchmark
use.  listed() names twelve of them, draw() gives further ones of the same ranges.

A case is one attention layer: `op` says what is called,
  step     the two calls of a decode step: append one token per sequence, then attend (query rotated)
  fused    the same step as one call, the query un-rotated (rap_decode_step_ex)
  attn     the attention call alone, over a cache that other code has filled
  draft    append n_new tokens per sequence, then attend for all of them at once (rap_decode_attn_multi)
  prefill  append n_new tokens per sequence, rotate their queries, causal attention (rap_prefill_attn_split)
`kind` is the element type of the cache (bf16, fp8, mx4), `page` the rows of a page (0: a dense cache).
Sequences have ctx rows after the call; with `ragged` their lengths are spread evenly between ctx / 16
and ctx and dealt out by the seed.  Values are i.i.d. N(0, 1), one K row in a hundred eight times as
long, which is what the repository's own workloads use in place of trained weights.
"""
import math

import numpy as np
import torch

import paper_2602_02599_amd as pkg

D_HEAD = 128
DEV = "cuda"


def _case(name, op, kind, batch, n_q, n_kv, pairs, d_v, ctx, n_new=1, ragged=False, page=0, theta=5.0e5):
    return {"name": name, "op": op, "kind": kind, "batch": batch, "n_q": n_q, "n_kv": n_kv, "pairs": pairs, "d_v": d_v,
            "ctx": ctx, "n_new": n_new, "ragged": ragged, "page": page, "theta": theta}


def listed():
    return [
        # one short conversation, 3B-sized layer: the smallest decode step, all launches and latency
        _case("one_short", "step", "bf16", 1, 24, 8, 45, 90, 2048),
        # one long conversation, 8B-sized layer, the step as one call
        _case("one_long", "fused", "bf16", 1, 32, 8, 45, 90, 32768),
        # the benchmark's own decode step: sixteen sequences of 8192 rows, append and attend
        _case("batch_step", "step", "bf16", 16, 32, 8, 45, 90, 8192),
        # a paged server: 64 sequences of mixed length, 128-row pages, the step as one call
        _case("paged_ragged", "fused", "bf16", 64, 32, 8, 45, 90, 16384, ragged=True, page=128),
        # few sequences of 131072 rows, five query heads per KV head, half the width
        _case("long_context", "attn", "bf16", 4, 40, 8, 32, 64, 131072, theta=1.0e6),
        # large batch over a wide cache whose V rows have an odd width
        _case("wide_odd", "attn", "bf16", 32, 32, 8, 58, 115, 32768, theta=1.0e6),
        # fp8 cache, the step as one call
        _case("fp8_step", "fused", "fp8", 32, 32, 8, 45, 90, 16384),
        # 4-bit cache, append and attend
        _case("mx4_step", "step", "mx4", 16, 32, 8, 45, 90, 32768),
        # four drafted tokens per sequence verified at once
        _case("draft_verify", "draft", "bf16", 16, 32, 8, 45, 90, 8192, n_new=4),
        # whole prompts of 8192 tokens: append, query rotation, causal attention
        _case("prefill", "prefill", "bf16", 8, 32, 8, 45, 90, 8192, n_new=8192),
        # chunked prefill: 512 tokens at the end of one long sequence
        _case("prefill_chunk", "prefill", "bf16", 1, 32, 8, 45, 90, 32768, n_new=512),
        # prompts of odd length into an fp8 cache of the wide layer
        _case("prefill_fp8_odd", "prefill", "fp8", 2, 32, 8, 58, 115, 4001, n_new=4001, theta=1.0e6),
    ]


def draw(rng):
    """One more case: op, cache kind, widths, heads, batch and length over the ranges of the listed ones."""
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    while True:
        op = rng.choice(["step", "fused", "attn", "draft", "prefill"])
        kind = rng.choice(["bf16", "bf16", "fp8"] + (["mx4"] if op in ("step", "attn") else []))
        n_kv, group = rng.choice([4, 8, 8]), rng.choice([3, 4, 4, 5, 8])
        pairs = rng.randint(24, 64)
        d_v = rng.choice([2 * pairs, rng.randint(48, 128)])
        page = rng.choice([0, 0, 128]) if kind != "mx4" else 0
        ragged = rng.random() < 0.4
        ctx, batch, n_new = log_int(500, 131072), log_int(1, 64), 1
        if op == "draft":
            n_new = rng.randint(2, 16 // group)
        if op == "prefill":
            ctx, batch = log_int(300, 16384), log_int(1, 16)
            n_new, ragged = rng.choice([ctx, log_int(16, min(ctx, 1024))]), False
        c = _case("", op, kind, batch, n_kv * group, n_kv, pairs, d_v, ctx, n_new, ragged, page, rng.choice([5.0e5, 1.0e6]))
        w, most = work(c), [work(x) for x in listed()]
        if w["bytes"] <= 0.9 * max(x["bytes"] for x in most) and w["flops"] <= 0.8 * max(x["flops"] for x in most):
            del c["name"]
            return c


# ---- sizes --------------------------------------------------------------------------------------

def _lens(case):
    """Rows of every sequence after the call, ascending."""
    b, ctx = case["batch"], case["ctx"]
    if not case["ragged"] or b == 1:
        return [ctx] * b
    lo = max(case["n_new"] + 1, ctx // 16)
    return [lo + (ctx - lo) * i // (b - 1) for i in range(b)]


def _row_bytes(case, d):
    """Bytes of one cache row of d elements (mx4: whole blocks of 32 codes and their scale bytes)."""
    blocks = (d + 31) // 32
    return {"bf16": 2 * d, "fp8": d, "mx4": 17 * blocks}[case["kind"]]


def work(case):
    d_k, d_v, n_q, n_kv, n = 2 * case["pairs"], case["d_v"], case["n_q"], case["n_kv"], case["n_new"]
    lens = _lens(case)
    rows = sum(lens)
    cache = n_kv * rows * (_row_bytes(case, d_k) + _row_bytes(case, d_v))
    tokens = case["batch"] * n
    new = 0 if case["op"] == "attn" else tokens * n_kv * 2 * (d_k + d_v)           # new rows, read
    query = tokens * n_q * 2 * d_k
    if case["op"] == "prefill":
        new += tokens * n_kv * (_row_bytes(case, d_k) + _row_bytes(case, d_v))      # cache rows written
        query *= 3                                                                  # read, written rotated, read
    out = tokens * n_q * 4 * d_v
    seen = sum(n * (m - n) + n * (n + 1) // 2 for m in lens)                        # visible (token, row) pairs
    return {"bytes": cache + new + query + out, "flops": 2 * (d_k + d_v) * n_q * seen}


# ---- inputs -------------------------------------------------------------------------------------

_E2M1 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]
_E2M1_MID = [0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0]


def _mx4_encode(x):
    """fp32 [..., d] -> (codes uint8 [..., 16 * blocks], scale bytes uint8 [..., 4])."""
    d = x.shape[-1]
    nb = (d + 31) // 32
    x = torch.nn.functional.pad(x, (0, 32 * nb - d)).unflatten(-1, (nb, 32))
    amax = x.abs().amax(-1, keepdim=True)
    e = torch.where(amax > 0, torch.frexp(amax).exponent - 3, torch.zeros((), dtype=torch.int32, device=x.device))
    y = torch.ldexp(x, -e)
    code = torch.bucketize(y.abs(), torch.tensor(_E2M1_MID, device=x.device)).to(torch.uint8) + 8 * (y < 0).to(torch.uint8)
    codes = (code[..., 0::2] | (code[..., 1::2] << 4)).flatten(-2)
    scales = torch.full(x.shape[:-2] + (4,), 127, dtype=torch.uint8, device=x.device)
    scales[..., :nb] = (e.squeeze(-1) + 127).to(torch.uint8)
    return codes.contiguous(), scales


def _mx4_decode(codes, scales, d):
    table = torch.tensor(_E2M1 + [-v for v in _E2M1], dtype=torch.float64, device=codes.device)
    v = torch.stack([table[(codes & 15).long()], table[(codes >> 4).long()]], -1).flatten(-2)
    s = torch.exp2(scales.double() - 127.0).repeat_interleave(32, -1)[..., : v.shape[-1]]
    return (v * s)[..., :d]


def _make(case, seed):
    """Every input of a case, from the seed alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    rng = np.random.default_rng(int(seed))
    B, n_kv, P, d_v, n = case["batch"], case["n_kv"], case["pairs"], case["d_v"], case["n_new"]
    lens = rng.permutation(np.array(_lens(case), dtype=np.int32))
    cap = -(-case["ctx"] // 128) * 128
    s = {"lens": torch.from_numpy(lens).to(DEV)}
    keep = np.stack([np.sort(rng.permutation(D_HEAD // 2)[:P]) for _ in range(n_kv)]).astype(np.int32)
    s["keep"] = torch.from_numpy(keep).to(DEV)
    first = lens - n
    s["pos"] = torch.from_numpy((first[:, None] + np.arange(n, dtype=np.int32)[None, :]).astype(np.int32)).to(DEV)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.bfloat16)

    page = case["page"]
    slabs = (B * (cap // page), n_kv, page) if page else (B, n_kv, cap)
    if page:
        order = torch.from_numpy(rng.permutation(slabs[0]).astype(np.int32)).to(DEV)
        s["table"] = order.view(B, cap // page).contiguous()
    for name, d, scale in (("k", 2 * P, 0.05), ("v", d_v, 0.02)):
        x = normal(*slabs, d)
        if name == "k":
            x *= torch.where(torch.rand(slabs, generator=g, device=DEV) < 0.01, 8.0, 1.0).to(torch.bfloat16)[..., None]
        if case["kind"] == "bf16":
            s[name] = x
        elif case["kind"] == "fp8":
            sc = scale * (1.0 + 0.25 * torch.rand((n_kv,), generator=g, device=DEV))
            s[name + "_scale"] = sc
            parts = [(p.float() / sc[:, None, None]).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8) for p in x.split(4 if not page else 64)]
            s[name] = torch.cat(parts)
        else:
            parts = [_mx4_encode(p.float()) for p in x.split(2)]
            s[name], s[name + "_scale"] = (torch.cat([p[i] for p in parts]) for i in (0, 1))
        del x
    s["k_new"], s["v_new"] = normal(B, n, n_kv, 2 * P), normal(B, n, n_kv, d_v)
    s["q"] = normal(B, n, case["n_q"], 2 * P)
    return s, cap


def prepare(case, seed):
    """The caches, the new tokens and queries, and what a program keeps beside them: the shape record,
    the block table, the workspace and the output buffer."""
    rap = pkg.load()
    s, cap = _make(case, seed)
    op, n, ctx = case["op"], case["n_new"], case["ctx"]
    s["rap"], s["case"], s["scale"] = rap, case, 1.0 / math.sqrt(D_HEAD)
    s["shape"] = rap.shape(case["batch"], case["n_q"], case["n_kv"], D_HEAD, case["pairs"], case["d_v"], cap, case["theta"])
    s["paging"] = rap.paging(case["page"], s["k"].shape[0], s["table"]) if case["page"] else None
    s["out"] = torch.empty((case["batch"], n, case["n_q"], case["d_v"]), dtype=torch.float32, device=DEV)
    if op == "prefill":
        need = rap.rap_prefill_attn_split_workspace_bytes(s["shape"], n, ctx)
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV) if need else None
        s["q_rot"] = torch.empty_like(s["q"])
    else:
        s["ws"] = rap.new_workspace(s["shape"], ctx, n_tok=n)
    return s


# ---- one pass -----------------------------------------------------------------------------------

def _append(s, n):
    r, a = s["rap"], (s["k_new"], s["v_new"], s["pos"], s["keep"], s["k"], s["v"])
    kind, pg = s["case"]["kind"], s["paging"]
    if kind == "mx4":
        r.rap_rope_append_mx4(s["shape"], n, s["k_new"], s["v_new"], s["pos"], s["keep"], s["k"], s["k_scale"], s["v"], s["v_scale"])
    elif kind == "fp8" and pg is not None:
        r.rap_rope_append_paged_q8(s["shape"], pg, n, *a, s["k_scale"], s["v_scale"])
    elif kind == "fp8":
        r.rap_rope_append_q8(s["shape"], n, *a, s["k_scale"], s["v_scale"])
    elif pg is not None:
        r.rap_rope_append_paged(s["shape"], pg, n, *a)
    else:
        r.rap_rope_append(s["shape"], n, *a)


def _attend(s):
    r, c, pg = s["rap"], s["case"], s["paging"]
    tail = (s["lens"], c["ctx"], s["out"], s["scale"], s["ws"])
    if c["kind"] == "mx4":
        r.rap_decode_attn_mx4(s["shape"], s["q"], s["k"], s["k_scale"], s["v"], s["v_scale"], *tail)
    elif c["kind"] == "fp8" and pg is not None:
        r.rap_decode_attn_paged_q8(s["shape"], pg, s["q"], None, None, s["k"], s["v"], s["k_scale"], s["v_scale"], *tail)
    elif c["kind"] == "fp8":
        r.rap_decode_attn_q8(s["shape"], s["q"], None, None, s["k"], s["v"], s["k_scale"], s["v_scale"], *tail)
    elif pg is not None:
        r.rap_decode_attn_paged(s["shape"], pg, s["q"], None, None, s["k"], s["v"], *tail)
    else:
        r.rap_decode_attn(s["shape"], s["q"], s["k"], s["v"], *tail)


def run(s):
    r, c = s["rap"], s["case"]
    op, n = c["op"], c["n_new"]
    scales = (s["k_scale"], s["v_scale"]) if c["kind"] == "fp8" else (None, None)
    if op == "attn":
        _attend(s)
        return {"out": s["out"]}
    done = {"out": s["out"], "k": s["k"], "v": s["v"]}
    if op == "step":
        _append(s, n)
        _attend(s)
    elif op == "fused":
        r.rap_decode_step_ex(s["shape"], s["k"], s["v"], *scales, s["paging"], s["k_new"], s["v_new"], s["pos"], s["keep"],
                             s["q"], False, s["lens"], c["ctx"], s["out"], s["scale"], s["ws"])
    elif op == "draft":
        _append(s, n)
        r.rap_decode_attn_multi(s["shape"], s["k"], s["v"], *scales, s["paging"], n, s["q"], s["lens"], c["ctx"], s["out"],
                                s["scale"], s["ws"])
    else:
        _append(s, n)
        r.rap_rope_queries(s["shape"], n, s["q"], s["pos"], s["keep"], s["q_rot"])
        r.rap_prefill_attn_split(s["shape"], s["k"], s["v"], *scales, s["paging"], n, s["q_rot"], s["lens"], c["ctx"],
                                 s["out"], s["scale"], s["ws"])
        done["q_rot"] = s["q_rot"]
    if c["kind"] == "mx4":
        done["k_scale"], done["v_scale"] = s["k_scale"], s["v_scale"]
    return done


# ---- what it should be --------------------------------------------------------------------------

def tolerance(case):
    """Outputs are fp32 sums of bf16 products with the probabilities held to 16 significant bits.  Against
    exact() the listed cases are 2.0e-6 to 3.0e-6 off, single values up to 1.3e-4; four times that.
    Cache codes stay the same."""
    return {"rel": 1.2e-5, "max": 5.2e-4}


def _rotate(x, pos, keep, theta, heads_per_row):
    """fp64 index-aware rotation of x [B, n, heads, 2P] at pos [B, n]."""
    P = x.shape[-1] // 2
    f = torch.pow(torch.tensor(theta, dtype=torch.float64, device=DEV), -2.0 * keep.double() / D_HEAD)
    phi = pos.double()[:, :, None, None] * f.repeat_interleave(heads_per_row, 0)
    a, b = x[..., :P].double(), x[..., P:].double()
    return torch.cat([a * torch.cos(phi) - b * torch.sin(phi), a * torch.sin(phi) + b * torch.cos(phi)], -1)


def _rounded(x, bits, low):
    """fp64 -> the nearest value of `bits` significant bits (ties to even), spaced 2^low at least."""
    m, e = torch.frexp(x)
    step = torch.clamp(e - bits, min=low)
    return torch.ldexp(torch.round(torch.ldexp(x, -step)), step)


def exact(case, seed):
    """The same in 64 bits: rotation, storage in the cache's own format, softmax attention per head."""
    s, cap = _make(case, seed)
    B, n_kv, n_q, n, d_k, d_v = case["batch"], case["n_kv"], case["n_q"], case["n_new"], 2 * case["pairs"], case["d_v"]
    G, kind, page, op = n_q // n_kv, case["kind"], case["page"], case["op"]
    lens = s["lens"].tolist()
    q = s["q"].double()
    done = {"out": None}
    k_rot = None
    if op != "attn":
        k_rot = _rotate(s["k_new"], s["pos"], s["keep"], case["theta"], 1)
        done["k"] = done["v"] = None
        if kind == "mx4":
            done["k_scale"] = done["v_scale"] = None
    if op in ("fused", "prefill"):
        q = _rotate(s["q"], s["pos"], s["keep"], case["theta"], G)
        if op == "prefill":
            done["q_rot"] = q
        q = _rounded(q, 8, -133)

    def slab(name, b, h, d):
        x = s[name]
        if page:
            x = x[s["table"][b].long(), h].reshape(cap, -1)
        else:
            x = x[b, h]
        if kind == "bf16":
            x = x.double()
        elif kind == "fp8":
            x = x.view(torch.float8_e4m3fn).float().double() * s[name + "_scale"][h].double()
        else:
            x = _mx4_decode(x, s[name + "_scale"][b, h], d)
        if k_rot is not None:
            new = (k_rot if name == "k" else s["v_new"].double())[b, :, h]
            if kind == "bf16":
                new = _rounded(new, 8, -133)
            elif kind == "fp8":
                sc = s[name + "_scale"][h].double()
                new = _rounded((new / sc).clamp(-448, 448), 4, -9) * sc
            else:
                codes, scales = _mx4_encode(new.float())
                new = _mx4_decode(codes, scales, d)
            x = x.clone()
            x[lens[b] - n : lens[b]] = new
        return x[: lens[b]]

    out = torch.empty((B, n, n_q, d_v), dtype=torch.float64, device=DEV)
    scale = 1.0 / math.sqrt(D_HEAD)
    for b in range(B):
        at = torch.arange(lens[b] - n, lens[b], device=DEV)
        seen = torch.arange(lens[b], device=DEV)[None, :] <= at[:, None]
        for h in range(n_kv):
            k, v = slab("k", b, h, d_k), slab("v", b, h, d_v)
            for a in range(h * G, (h + 1) * G):
                x = (q[b, :, a] @ k.t()) * scale
                x.masked_fill_(~seen, -math.inf)
                out[b, :, a] = torch.softmax(x, -1) @ v
    done["out"] = out
    return done
