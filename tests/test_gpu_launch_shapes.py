"""Kernels and dispatch rules at the sizes where they can go wrong: every instantiation width of the
prefill kernel with the cache ending inside its last row, range counts at the edges of the combining
kernel's groups, block counts of 4-bit rows, the ranges the split plan picks, and workspaces of the
size the plain range rule asks for.  Against the float64 oracle; bars as in tests/helpers.py."""
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
    print("[launch shapes] " + msg, flush=True)


def _caches(rap, rng, B, Hkv, cap, P, dv, lens, fp8, page_rows):
    k = rng.standard_normal((B, Hkv, cap, 2 * P))
    v = rng.standard_normal((B, Hkv, cap, dv))
    ks = (rng.uniform(4.0, 6.0, Hkv) / 448.0).astype(np.float32) if fp8 else None
    vs = (rng.uniform(4.0, 6.0, Hkv) / 448.0).astype(np.float32) if fp8 else None
    return H.encode_cache(rap, rng, k, v, lens, fp8, page_rows, ks, vs) + (ks, vs)


# d_k in every quarter (one to four steps of 32), d_v in every sixteenth and odd ones; pages of 64
# rows, and dense caches that end with the last row of the last sequence, whose last piece then takes
# the loads of single dwords or bytes (that no load leaves the cache is a CPU test of the load plan)
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("P,dv,Hq,Hkv,n_new,page_rows", [
    (1, 1, 2, 2, 65, 0), (9, 16, 8, 8, 33, 0), (16, 17, 4, 4, 70, 64), (17, 32, 16, 8, 64, 0), (24, 45, 3, 1, 129, 0),
    (32, 48, 8, 8, 47, 64), (33, 64, 10, 2, 52, 0), (35, 66, 4, 4, 96, 0), (45, 79, 8, 2, 31, 64), (48, 80, 4, 2, 64, 0),
    (45, 96, 16, 1, 40, 0), (49, 97, 4, 4, 61, 0), (51, 102, 8, 8, 35, 64), (58, 112, 6, 2, 63, 0), (61, 113, 4, 4, 90, 0),
    (64, 127, 8, 8, 20, 64), (64, 128, 8, 4, 65, 0)])
def test_prefill_widths(rap, fp8, P, dv, Hq, Hkv, n_new, page_rows):
    """Whole and cut into key ranges, over a cache that holds exactly the rows of the longest sequence."""
    _say("prefill P=%d dv=%d heads %d/%d n_new=%d fp8=%s pages=%d" % (P, dv, Hq, Hkv, n_new, fp8, page_rows))
    cap = 576
    lens = np.asarray([cap - 41, cap], dtype=np.int64)         # the last sequence fills its slab, the last of the cache
    rng = np.random.Generator(np.random.PCG64(7000 + P + dv))
    kd, vd, kdev, vdev, ksd, vsd, pg, ks, vs = _caches(rap, rng, 2, Hkv, cap, P, dv, lens, fp8, page_rows)
    qb = O.f64_to_bf16_bits_rne(rng.standard_normal((2, n_new, Hq, 2 * P)))
    q, sl = I.from_bits(qb, DEV), torch.from_numpy(lens.astype(np.int32)).to(DEV)
    scale = 1.0 / math.sqrt(2 * P)
    shp = rap.shape(2, Hq, Hkv, 128, P, dv, cap, 5e5)
    guard, out = H.guarded_out((2, n_new, Hq, dv), DEV)
    rap.rap_prefill_attn_ex(shp, kdev, vdev, ksd, vsd, pg, n_new, q, sl, cap, out, scale)
    torch.cuda.synchronize()
    guard.check("out of rap_prefill_attn_ex")
    ref = O.prefill_attn_q8_ref(qb, kd, vd, ks, vs, lens, scale) if fp8 else O.prefill_attn_ref(qb, kd, vd, lens, scale)
    H.assert_attn_close(out.cpu().numpy(), ref, "prefill")
    need = rap.rap_prefill_attn_split_workspace_bytes(shp, n_new, cap)
    if need:
        gw = H.Guarded(need, DEV)
        cut = torch.full_like(out, float("nan"))
        rap.rap_prefill_attn_split(shp, kdev, vdev, ksd, vsd, pg, n_new, q, sl, cap, cut, scale, gw.bytes)
        torch.cuda.synchronize()
        gw.check("workspace of rap_prefill_attn_split")
        H.assert_attn_close(cut.cpu().numpy(), ref, "prefill in key ranges")


# eight slots per thread and round; one, two, four or eight groups of threads; loops over one, up to four,
# up to eight and up to sixteen new tokens
@pytest.mark.parametrize("n_tok", [1, 2, 5, 11])
@pytest.mark.parametrize("n_split", [7, 8, 9, 16, 17, 32, 33, 64, 65, 130])
def test_range_counts(rap, n_split, n_tok):
    """Ranges of 128 rows up to more than the combining kernel's groups read at once: full sequences,
    one that leaves the last ranges empty, an empty one (NaN in every slot of the workspace)."""
    P, dv, Hq, Hkv = 10, 21, 3 if n_tok <= 5 else 1, 1
    cap = 128 * n_split
    lens = np.asarray([cap, cap - 128 * (n_split // 3) - 5, 0, cap - 1], dtype=np.int64)
    _say("ranges %d tokens %d" % (n_split, n_tok))
    rng = np.random.Generator(np.random.PCG64(900 + n_split))
    kd, vd, kdev, vdev, _, _, _, _, _ = _caches(rap, rng, 4, Hkv, cap, P, dv, lens, False, 0)
    qb = O.f64_to_bf16_bits_rne(rng.standard_normal((4, n_tok, Hq, 2 * P)))
    q, sl = I.from_bits(qb, DEV), torch.from_numpy(lens.astype(np.int32)).to(DEV)
    shp, scale = rap.shape(4, Hq, Hkv, 128, P, dv, cap, 5e5), 0.25
    tun = rap.tuning(rows_per_split=128)
    gw, ws = H.guarded_workspace(rap, shp, cap, tun, n_tok=n_tok)
    go, out = H.guarded_out((4, n_tok, Hq, dv), DEV)
    rap.rap_decode_attn_multi(shp, kdev, vdev, None, None, None, n_tok, q, sl, cap, out, scale, ws, tun)
    torch.cuda.synchronize()
    gw.check("workspace")
    go.check("out")
    H.assert_attn_close(out.cpu().numpy(), O.prefill_attn_ref(qb, kd, vd, lens, scale), "%d ranges" % n_split)


# around the numbers of 16-token runs up to which they are four tokens long: 1536 (bf16 append), 3584 (fp8), 1024 (queries)
@pytest.mark.parametrize("n_new", [1024, 1025, 1536, 1537, 3584, 3591])
def test_bulk_run_lengths(rap, n_new):
    """A prefill-sized append and rotation as one call against the same tokens in calls of 48, which take the short runs
    (an oracle test of their own): bit for bit, with a jump in the positions and rows that are skipped."""
    P, dv, H16 = 9, 11, 16
    cap = (n_new + 200 + 15) // 16 * 16
    _say("bulk runs n_new=%d" % n_new)
    g = torch.Generator(device=DEV); g.manual_seed(n_new)
    rand = lambda *s: torch.randn(s, generator=g, device=DEV).to(torch.bfloat16)
    kn, vn, q = rand(1, n_new, H16, 2 * P), rand(1, n_new, H16, dv), rand(1, n_new, 2 * H16, 2 * P)
    pos = torch.arange(n_new, dtype=torch.int32, device=DEV)
    pos[n_new // 2:] += 101
    pos[5] = -1
    pos = pos[None].contiguous()
    keep = torch.arange(P, dtype=torch.int32, device=DEV).repeat(H16, 1).contiguous()
    sc = torch.rand(H16, generator=g, device=DEV) * 0.02 + 0.01
    shp = rap.shape(1, 2 * H16, H16, 128, P, dv, cap, 5e5)
    done = []
    for step in (n_new, 48):
        k, v, k8, v8 = (torch.zeros((1, H16, cap, d), dtype=t, device=DEV) for t in (torch.bfloat16, torch.uint8) for d in (2 * P, dv))
        rot = torch.empty_like(q)
        for at in range(0, n_new, step):
            n = min(step, n_new - at)
            part = lambda x: x[:, at:at + n].contiguous()
            rap.rap_rope_append(shp, n, part(kn), part(vn), part(pos), keep, k, v)
            rap.rap_rope_append_q8(shp, n, part(kn), part(vn), part(pos), keep, k8, v8, sc, sc)
            piece = torch.empty_like(part(q))
            rap.rap_rope_queries(shp, n, part(q), part(pos), keep, piece)
            rot[:, at:at + n] = piece
        torch.cuda.synchronize()
        done.append((k, v, k8, v8, rot))
    for x, y in zip(*done):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))


# lengths of a batch in units of its longest: all full, all alike but shorter, spread out, empty and single-row ones among
# long ones, one long one
LENGTHS = {"full": lambda i, B: 1.0, "alike": lambda i, B: 0.6, "spread": lambda i, B: (i + 1) / B,
           "gaps": lambda i, B: (0.0, 1.0, 1e-9, 0.37)[i % 4], "one": lambda i, B: 1.0 if i == B - 1 else 0.02}


@pytest.mark.parametrize("kind", ["bf16", "fp8", "mx4", "paged"])
@pytest.mark.parametrize("B,ctx,Hq,Hkv", [(40, 3000, 16, 8), (9, 9000, 8, 8), (3, 50000, 16, 8), (64, 3100, 12, 4), (2, 60000, 15, 3)])
def test_ranges_by_length(rap, kind, B, ctx, Hq, Hkv):
    """The automatic ranges, which follow the lengths, against ranges of a fixed number of rows, for every pattern of
    lengths: plain attention, several tokens, the one-call step (its new row last, in the middle, nowhere)."""
    P, dv, cap = 6, 10, (ctx + 127) // 128 * 128
    fixed = rap.tuning(rows_per_split=4096)
    g = torch.Generator(device=DEV); g.manual_seed(B)
    rand = lambda *s: torch.randn(s, generator=g, device=DEV)
    rows = (B * (cap // 128), Hkv, 128) if kind == "paged" else (B, Hkv, cap)
    shp, scale = rap.shape(B, Hq, Hkv, 128, P, dv, cap, 5e5), 0.3
    ks = vs = pg = None
    if kind == "mx4":
        k, v = (torch.randint(0, 256, rows + (16,), generator=g, device=DEV, dtype=torch.int32).to(torch.uint8) for _ in range(2))
        sc = torch.randint(123, 128, rows + (4,), generator=g, device=DEV, dtype=torch.int32).to(torch.uint8)
    else:
        k, v = rand(*rows, 2 * P).to(torch.bfloat16), rand(*rows, dv).to(torch.bfloat16)
        if kind == "fp8":
            k, v = (x.to(torch.float8_e4m3fn).view(torch.uint8) for x in (k, v))
            ks, vs = (torch.rand(Hkv, generator=g, device=DEV) + 0.5 for _ in range(2))
        if kind == "paged":
            pg = rap.paging(128, rows[0], torch.randperm(rows[0], generator=g, device=DEV).to(torch.int32).view(B, -1).contiguous())
    keep = torch.arange(P, dtype=torch.int32, device=DEV).repeat(Hkv, 1).contiguous()

    def both(shape, call, n_tok=1):
        outs = []
        for tun in (None, fixed):
            gw, ws = H.guarded_workspace(rap, shp, ctx, tun, n_tok=n_tok)
            go, out = H.guarded_out(shape, DEV)
            call(out, ws, tun)
            torch.cuda.synchronize()
            gw.check("workspace")
            go.check("out")
            outs.append(out)
        assert not torch.isnan(outs[0]).any()
        worst = ((outs[0] - outs[1]).abs().max() / outs[1].abs().max()).item()
        assert worst < 2e-5, worst                      # sums of 16-bit probabilities, in another order

    for name, f in LENGTHS.items():
        _say("by length %s B=%d ctx=%d %s" % (kind, B, ctx, name))
        lens = torch.tensor([min(ctx, int(math.ceil(ctx * f(i, B)))) for i in range(B)], dtype=torch.int32)
        lens = lens[torch.randperm(B, generator=torch.Generator().manual_seed(7))].to(DEV)
        if kind == "mx4":
            q = rand(B, Hq, 2 * P).to(torch.bfloat16)
            both((B, Hq, dv), lambda o, w, t: rap.rap_decode_attn_mx4(shp, q, k, sc, v, sc, lens, ctx, o, scale, w, t))
            continue
        for n_tok in (1, 2, 3):
            q = rand(B, n_tok, Hq, 2 * P).to(torch.bfloat16)
            both((B, n_tok, Hq, dv), lambda o, w, t: rap.rap_decode_attn_multi(shp, k, v, ks, vs, pg, n_tok, q, lens, ctx, o, scale, w, t), n_tok)
        q1, k1, v1 = rand(B, Hq, 2 * P).to(torch.bfloat16), rand(B, Hkv, 2 * P).to(torch.bfloat16), rand(B, Hkv, dv).to(torch.bfloat16)
        for at in ("last", "middle", "nowhere"):
            pos = (lens - 1 if at == "last" else lens // 2 if at == "middle" else lens * 0 - 1).to(torch.int32)
            both((B, Hq, dv), lambda o, w, t: rap.rap_decode_step_ex(shp, k, v, ks, vs, pg, k1, v1, pos, keep, q1, False, lens, ctx, o, scale, w, t))


# one, two, four or eight sets of lanes per query row; channels in fours, with a last four that overlaps, fewer than four
@pytest.mark.parametrize("rows,dv", [(2048, 90), (2049, 1), (4096, 3), (4100, 4), (8192, 5), (8200, 128), (16640, 127)])
def test_prefill_range_counts(rap, rows, dv):
    """A few tokens at the end of sequences in ranges of 256 rows, up to more ranges than the combining kernel reads
    at once: a full sequence, one that leaves the last ranges empty, one shorter than the chunk (NaN in every slot)."""
    P, Hq, Hkv, n_new, cap = 9, 3, 1, 5, (rows + 15) // 16 * 16
    lens = np.asarray([rows, rows - rows // 3, 2], dtype=np.int64)
    _say("prefill ranges rows=%d dv=%d" % (rows, dv))
    rng = np.random.Generator(np.random.PCG64(1900 + rows))
    kd, vd, kdev, vdev, _, _, _, _, _ = _caches(rap, rng, 3, Hkv, cap, P, dv, lens, False, 0)
    qb = O.f64_to_bf16_bits_rne(rng.standard_normal((3, n_new, Hq, 2 * P)))
    q, sl = I.from_bits(qb, DEV), torch.from_numpy(lens.astype(np.int32)).to(DEV)
    shp, scale = rap.shape(3, Hq, Hkv, 128, P, dv, cap, 5e5), 0.25
    need = rap.rap_prefill_attn_split_workspace_bytes(shp, n_new, rows)
    gw, (go, out) = H.Guarded(need, DEV), H.guarded_out((3, n_new, Hq, dv), DEV)
    gw.bytes.fill_(0xFF)
    rap.rap_prefill_attn_split(shp, kdev, vdev, None, None, None, n_new, q, sl, rows, out, scale, gw.bytes)
    torch.cuda.synchronize()
    gw.check("workspace")
    go.check("out")
    H.assert_attn_close(out.cpu().numpy(), O.prefill_attn_ref(qb, kd, vd, lens, scale), "%d rows in ranges" % rows)


@pytest.mark.parametrize("P,dv", [(16, 65), (5, 128), (17, 32), (30, 96), (32, 97), (40, 31), (48, 64), (45, 128), (49, 1), (64, 33), (56, 95)])
def test_mx4_block_counts(rap, P, dv):
    """4-bit rows with every pairing of one to four K and V blocks, sequence lengths at the edges of the
    32-row tile: bit for bit the bf16 call on the dequantised cache, and the oracle."""
    _say("mx4 P=%d dv=%d" % (P, dv))
    lens = np.asarray([1, 31, 32, 33, 128, 161], dtype=np.int64)
    B, Hkv, Hq, cap = len(lens), 2, 6, 168
    rng = np.random.Generator(np.random.PCG64(5 + P + dv))
    kc, ks = O.mx4_quantize_rows(rng.standard_normal((B, Hkv, cap, 2 * P)))
    vc, vs = O.mx4_quantize_rows(rng.standard_normal((B, Hkv, cap, dv)))
    for b in range(B):
        for x in (kc, ks, vc, vs):
            x[b, :, int(lens[b]):] = 0xFF
    qb = O.f64_to_bf16_bits_rne(rng.standard_normal((B, Hq, 2 * P)))
    dev = [torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in (kc, ks, vc, vs)]
    q, sl = I.from_bits(qb, DEV), torch.from_numpy(lens.astype(np.int32)).to(DEV)
    shp, scale = rap.shape(B, Hq, Hkv, 128, P, dv, cap, 5e5), 1.0 / math.sqrt(2 * P)
    ref = O.attn_mx4_ref(qb, kc, ks, vc, vs, lens, scale, 2 * P, dv)
    kb = I.from_bits(O.f64_to_bf16_bits_rne(np.nan_to_num(O.mx4_dequantize_rows(kc, ks, 2 * P))), DEV)
    vb = I.from_bits(O.f64_to_bf16_bits_rne(np.nan_to_num(O.mx4_dequantize_rows(vc, vs, dv))), DEV)
    for rps in (0, 128):
        tun = rap.tuning(rows_per_split=rps)
        gw, ws = H.guarded_workspace(rap, shp, cap, tun)
        go, out = H.guarded_out((B, Hq, dv), DEV)
        rap.rap_decode_attn_mx4(shp, q, *dev, sl, cap, out, scale, ws, tun)
        torch.cuda.synchronize()
        gw.check("workspace")
        go.check("out")
        H.assert_attn_close(out.cpu().numpy(), ref, "mx4")
        b16 = torch.empty_like(out)
        rap.rap_decode_attn(shp, q, kb, vb, sl, cap, b16, scale, ws, tun)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int32), b16.view(torch.int32)), "differs from the bf16 call on the dequantised cache"


def _slots_bytes(B, Hq, dv, n_split):
    """Workspace of n_split ranges as rap_decode_attn lays it out: accumulators, (reference, sum) pairs."""
    up = lambda x: (x + 255) // 256 * 256
    return up(B * Hq * (n_split + 1) * dv * 4) + up(B * Hq * (n_split + 1) * 8) + 256


@pytest.mark.parametrize("B,ctx,plan,plain", [(1, 512, 4, 1), (1, 2048, 16, 4), (2, 384, 1, 1), (3, 5000, 10, 10), (1, 130, 1, 1), (24, 1100, 2, 2), (32, 1024, 1, 2), (14, 790, 2, 2)])
def test_plan_and_smaller_workspace(rap, B, ctx, plan, plain):
    """The ranges of the automatic plan at few sequences and ragged lengths, and the same call with a
    workspace that only holds the plain rule's ranges (none where that is a single range); what the
    library asks for is never less than the latter, also where the plan keeps rows whole (32 x 1024)."""
    P, dv, Hq, Hkv = 20, 40, 8, 8
    cap = (ctx + 7) // 8 * 8
    _say("plan B=%d ctx=%d" % (B, ctx))
    rng = np.random.Generator(np.random.PCG64(40 + ctx))
    lens = rng.integers(1, ctx + 1, B).astype(np.int64)
    lens[0] = ctx
    kd, vd, kdev, vdev, _, _, _, _, _ = _caches(rap, rng, B, Hkv, cap, P, dv, lens, False, 0)
    qb = O.f64_to_bf16_bits_rne(rng.standard_normal((B, Hq, 2 * P)))
    q, sl = I.from_bits(qb, DEV), torch.from_numpy(lens.astype(np.int32)).to(DEV)
    shp, scale = rap.shape(B, Hq, Hkv, 128, P, dv, cap, 5e5), 0.2
    ref = O.attn_ref(qb, kd, vd, lens, scale)
    gw, ws = H.guarded_workspace(rap, shp, ctx)
    small = H.Guarded(_slots_bytes(B, Hq, dv, plain), DEV) if plain > 1 else None
    for which, g, w in (("planned", gw, ws), ("plain", small, small.bytes if small else None)):
        go, out = H.guarded_out((B, Hq, dv), DEV)
        rap.rap_decode_attn(shp, q, kdev, vdev, sl, ctx, out, scale, w)
        torch.cuda.synchronize()
        go.check("out")
        if g is not None:
            g.check("workspace")
        H.assert_attn_close(out.cpu().numpy(), ref, which)
        n = plan if which == "planned" else min(plan, plain)
        if g is not None and n > 1:                            # the first sequence is full: every range left its reference and sum
            at = (B * Hq * (n + 1) * dv * 4 + 255) // 256 * 256
            ml = w[at:at + B * Hq * n * 8].view(torch.float32).view(B * Hq, n, 2)
            assert not torch.isnan(ml[:Hq]).any(), "%d ranges expected" % n
        elif g is not None:                                    # a single range stores the output itself
            assert bool((w == 0xFF).all()), "no ranges expected"
    if plain > 1:                                              # one byte less is refused
        assert ws.numel() >= max(_slots_bytes(B, Hq, dv, plan), small.bytes.numel())
        assert rap.rap_decode_attn(shp, q, kdev, vdev, sl, ctx, out, scale, small.bytes[:-1], check=False) == 5
