"""Decode attention whose row ranges follow the lengths of the batch, at real widths against the float64 oracle, and what
the header says of the order of the sums: with ranges of a fixed number of rows a sequence's output does not depend on
its neighbours.  Bars as in tests/helpers.py."""
import math

import numpy as np
import pytest
import torch

from oracle import rap_oracle as O
import rap_inputs as I
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _say(msg):
    print("[by length] " + msg, flush=True)


class Cache:
    """A cache of random rows; those at and beyond lens[b], and unused pages, hold NaN patterns."""

    def __init__(self, rap, kind, P, dv, Hkv, cap, lens, seed):
        B = len(lens)
        self.kind, self.P, self.dv, self.cap, self.lens = kind, P, dv, cap, lens
        self.g = g = torch.Generator(device=DEV)
        g.manual_seed(seed)
        self.scales, self.pg, self.table = (None, None), None, None
        dense = []
        for d in (2 * P, dv):
            if kind == "mx4":
                x = torch.randint(0, 256, (B, Hkv, cap, 16 * ((d + 31) // 32)), generator=g, device=DEV, dtype=torch.int32).to(torch.uint8)
                s = torch.randint(123, 128, (B, Hkv, cap, 4), generator=g, device=DEV, dtype=torch.int32).to(torch.uint8)
                for b in range(B):
                    x[b, :, lens[b]:] = s[b, :, lens[b]:] = 0xFF
                self.scales += (s,)
            else:
                x = torch.randn((B, Hkv, cap, d), generator=g, device=DEV, dtype=torch.bfloat16)
                if kind.startswith("fp8"):
                    x = (64.0 * x).to(torch.float8_e4m3fn).view(torch.uint8)
                    self.scales += ((torch.rand(Hkv, generator=g, device=DEV) + 0.5) / 64.0,)
                for b in range(B):
                    if x.dtype == torch.uint8:
                        x[b, :, lens[b]:] = 0x7F
                    else:
                        x[b, :, lens[b]:] = float("nan")
            dense.append(x)
        if len(self.scales) > 2:
            self.scales = self.scales[2:]
        if kind.endswith("paged"):
            n = B * cap // 128
            self.table = torch.randperm(n + 2, generator=g, device=DEV)[:n]
            self.pg = rap.paging(128, n + 2, self.table.to(torch.int32).view(B, -1).contiguous())
            pools = []
            for x in dense:
                pool = torch.full((n + 2, Hkv, 128, x.shape[-1]), 0x7F if x.dtype == torch.uint8 else float("nan"), dtype=x.dtype, device=DEV)
                pool[self.table] = x.view(B, Hkv, -1, 128, x.shape[-1]).transpose(1, 2).flatten(0, 1)
                pools.append(pool)
            dense = pools
        self.k, self.v = dense

    def head(self, h, seqs):
        """K and V of KV head h of some sequences, for the oracle: [len(seqs), 1, cap, d] bit patterns."""
        out = []
        for x in (self.k, self.v):
            if self.pg is not None:
                x = x[self.table].view(len(self.lens), -1, *x.shape[1:])[seqs][:, :, h].flatten(1, 2)
            else:
                x = x[seqs][:, h]
            x = x[:, None].contiguous()
            out.append(x.cpu().numpy() if x.dtype == torch.uint8 else I.bits(x))
        return out

    def reference(self, q, h, seqs, scale):
        """q [B, n_tok, H_q, d_k] -> the oracle's rows of KV head h, [len(seqs), n_tok, G, d_v]."""
        G = q.shape[2] // self.k.shape[1]
        qb = I.bits(q[seqs][:, :, h * G:(h + 1) * G].contiguous())
        k, v = self.head(h, seqs)
        lens = [self.lens[b] for b in seqs]
        if self.kind == "mx4":
            ks, vs = (s[seqs][:, h:h + 1].cpu().numpy() for s in self.scales)
            return O.attn_mx4_ref(qb[:, 0], k, ks, v, vs, lens, scale, 2 * self.P, self.dv)[:, None]
        if self.kind.startswith("fp8"):
            ks, vs = (s[h:h + 1].cpu().numpy() for s in self.scales)
            return O.prefill_attn_q8_ref(qb, k, v, ks, vs, lens, scale)
        return O.prefill_attn_ref(qb, k, v, lens, scale)


# 9 x 9000 rows over 8 KV heads: 512 workgroups of about 1400 rows.  One to four score steps, channel tiles in pairs and
# not, with a lean loop and without (33 pairs, d_v = 100)
WIDTHS = [(45, 90), (33, 100), (58, 115), (64, 128), (30, 61)]
LENS = {"spread": lambda i: 600 + 8400 * i // 8, "alike": lambda i: 9000 - 97 * (i * 5 % 9), "few long": lambda i: 9000 if i in (2, 7) else 300 + i}


@pytest.mark.parametrize("kind", ["bf16", "paged", "fp8", "fp8 paged", "mx4"])
@pytest.mark.parametrize("P,dv", WIDTHS)
def test_real_widths_against_the_oracle(rap, kind, P, dv):
    B, Hkv, Hq, cap, ctx = 9, 8, 32, 9088, 9000
    for n, (name, length) in enumerate(LENS.items()):
        _say("%s P=%d dv=%d lengths %s" % (kind, P, dv, name))
        lens = [length((i * 4 + n) % 9) for i in range(B)]
        c = Cache(rap, kind, P, dv, Hkv, cap, lens, 31 * P + n)
        shp, scale = rap.shape(B, Hq, Hkv, 128, P, dv, cap, 5e5), (0.2 if kind == "mx4" else 1.0) / math.sqrt(2 * P)
        sl = torch.tensor(lens, dtype=torch.int32, device=DEV)
        h = (P + dv + n) % Hkv
        order = sorted(range(B), key=lambda b: lens[b])
        seqs = [order[0], order[4], order[8]]
        for n_tok in (1,) if kind == "mx4" else (1, 3):
            q = torch.randn((B, n_tok, Hq, 2 * P), generator=c.g, device=DEV, dtype=torch.bfloat16)
            gw, ws = H.guarded_workspace(rap, shp, ctx, n_tok=n_tok)
            go, out = H.guarded_out((B, n_tok, Hq, dv), DEV)
            if kind == "mx4":
                rap.rap_decode_attn_mx4(shp, q, c.k, c.scales[0], c.v, c.scales[1], sl, ctx, out, scale, ws)
            else:
                rap.rap_decode_attn_multi(shp, c.k, c.v, *c.scales, c.pg, n_tok, q, sl, ctx, out, scale, ws)
            torch.cuda.synchronize()
            gw.check("workspace")
            go.check("out")
            assert bool(torch.isfinite(out).all())
            H.assert_attn_close(out[seqs][:, :, 4 * h:4 * h + 4].cpu().numpy(), c.reference(q, h, seqs, scale), "%s, %d tokens" % (name, n_tok))
        if kind == "mx4":
            continue
        # the one-call step: its new row replaces the last one
        rand = lambda *s: torch.randn(s, generator=c.g, device=DEV, dtype=torch.bfloat16)
        q, kn, vn = rand(B, Hq, 2 * P), rand(B, Hkv, 2 * P), rand(B, Hkv, dv)
        keep = torch.arange(P, dtype=torch.int32, device=DEV).repeat(Hkv, 1).contiguous()
        gw, ws = H.guarded_workspace(rap, shp, ctx)
        go, out = H.guarded_out((B, Hq, dv), DEV)
        rap.rap_decode_step_ex(shp, c.k, c.v, *c.scales, c.pg, kn, vn, sl - 1, keep, q, True, sl, ctx, out, scale, ws)
        torch.cuda.synchronize()
        gw.check("workspace")
        go.check("out")
        H.assert_attn_close(out[seqs][:, None, 4 * h:4 * h + 4].cpu().numpy(), c.reference(q[:, None], h, seqs, scale), name + ", one call")


@pytest.mark.parametrize("name", list(LENS))
def test_extreme_scores(rap, name):
    """One row that outweighs all others (first, last, in the middle of a sequence), rows that all weigh the same at a score far
    below zero, and a NaN in one row of one KV head, whose rows are zeros while all others keep their bits."""
    B, Hkv, Hq, P, dv, cap, ctx = 9, 8, 32, 45, 90, 9088, 9000
    lens = [LENS[name]((i * 4) % 9) for i in range(B)]
    _say("extreme scores, lengths %s" % name)
    c = Cache(rap, "bf16", P, dv, Hkv, cap, lens, 77)
    shp, scale = rap.shape(B, Hq, Hkv, 128, P, dv, cap, 5e5), 1.0 / math.sqrt(2 * P)
    sl = torch.tensor(lens, dtype=torch.int32, device=DEV)
    q = torch.randn((B, Hq, 2 * P), generator=c.g, device=DEV, dtype=torch.bfloat16)

    def attend():
        gw, ws = H.guarded_workspace(rap, shp, ctx)
        go, out = H.guarded_out((B, Hq, dv), DEV)
        rap.rap_decode_attn(shp, q, c.k, c.v, sl, ctx, out, scale, ws)
        torch.cuda.synchronize()
        gw.check("workspace")
        go.check("out")
        return out.clone()

    h = 3
    for b in range(B):
        c.k[b, h, [0, lens[b] - 1, lens[b] // 2][b % 3]] = 40.0 * q[b, 4 * h + 1]
        c.k[b, h + 1, :lens[b]] = -40.0 * q[b, 4 * h + 6]
    out = attend()
    assert bool(torch.isfinite(out).all())
    for b in range(B):
        row = c.v[b, h, [0, lens[b] - 1, lens[b] // 2][b % 3]].float()
        # a score some 340 above the others leaves them exp(-340); one probability in head and remainder is exact
        assert torch.equal(out[b, 4 * h + 1], row)
        mean = c.v[b, h + 1, :lens[b]].double().mean(0)
        # fp32 sums of up to 9000 values of order one, over their number: 1e-7 of their root mean square each
        assert (out[b, 4 * h + 6].double() - mean).abs().max().item() < 1e-6
    bad = 5
    c.k[bad, 6, lens[bad] // 3, 7] = float("nan")
    nan = attend()
    assert bool((nan[bad, 24:28] == 0).all())
    nan[bad, 24:28] = out[bad, 24:28]
    assert torch.equal(nan.view(torch.int32), out.view(torch.int32))


@pytest.mark.parametrize("kind", ["bf16", "fp8", "paged"])
def test_fixed_ranges_do_not_depend_on_neighbours(rap, kind):
    """24 sequences whose ranges would follow their lengths: with rows_per_split set, and with a workspace that only holds the
    plainer rule's ranges (two of 4096 rows), an output row keeps its bits when the other sequences' lengths change."""
    B, Hkv, Hq, P, dv, ctx = 24, 8, 8, 20, 41, 8192
    c = Cache(rap, kind, P, dv, Hkv, ctx, [ctx] * B, 5)
    shp = rap.shape(B, Hq, Hkv, 128, P, dv, ctx, 5e5)
    up = lambda x: (x + 255) // 256 * 256
    plain = up(B * Hq * 3 * dv * 4) + up(B * Hq * 3 * 8) + 256
    assert plain < rap.rap_decode_attn_workspace_bytes(shp, ctx, None)
    rand = lambda *s: torch.randn(s, generator=c.g, device=DEV, dtype=torch.bfloat16)
    q, kn, vn = rand(B, Hq, 2 * P), rand(B, Hkv, 2 * P), rand(B, Hkv, dv)
    keep = torch.arange(P, dtype=torch.int32, device=DEV).repeat(Hkv, 1).contiguous()
    kept = {1: 5001, 13: 8192, 22: 130}
    for rows in (1024, 0):
        tun = rap.tuning(rows_per_split=rows)
        size = rap.rap_decode_attn_workspace_bytes(shp, ctx, tun) if rows else plain
        seen = []
        for f in (lambda i: ctx, lambda i: 1 + (ctx - 1) * i // (B - 1), lambda i: 257, lambda i: ctx - 128 * (i % 3)):
            _say("%s, neighbours change, rows_per_split %d" % (kind, rows))
            sl = torch.tensor([kept.get(i, f(i)) for i in range(B)], dtype=torch.int32, device=DEV)
            one, step = (torch.empty((B, Hq, dv), dtype=torch.float32, device=DEV) for _ in range(2))
            ws = torch.full((size,), 0xFF, dtype=torch.uint8, device=DEV)
            rap.rap_decode_attn_multi(shp, c.k, c.v, *c.scales, c.pg, 1, q, sl, ctx, one, 0.2, ws, tun)
            k, v = c.k.clone(), c.v.clone()
            rap.rap_decode_step_ex(shp, k, v, *c.scales, c.pg, kn, vn, sl - 1, keep, q, True, sl, ctx, step, 0.2, ws, tun)
            torch.cuda.synchronize()
            seen.append(torch.stack([x[list(kept)] for x in (one, step)]).view(torch.int32))
        for x in seen[1:]:
            assert torch.equal(seen[0], x)
