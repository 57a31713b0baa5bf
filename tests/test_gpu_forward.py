"""GPU parity of the target forward (Alg. 1 Step 3) against the CPU oracle,
through the C ABI.

float32 configuration: max |logit error| <= 1e-4.
bf16 configurations: the oracle rounds to bf16 at the same tensor boundaries as
the device; every pass is held to the oracle's own rounding noise (see
tests.gpu_util.check_bf16_logits): bf16 rounding makes the forward chaotic, and
the stated max |logit error| <= 2e-2 lies below that noise except for shallow
models at the small width, where it is asserted as well."""
import numpy as np
import pytest
import torch

import paper_2601_05149_amd as mulo
from oracle import decoder as OD
from tests.gpu_util import (DEV, TILES, check_bf16_logits, dev, device_weights, make_ctx, make_ctx_from_device, say, tiles_of)
from workloads import configs as WC
from workloads import generators as G

pytestmark = pytest.mark.gpu

from tests.cases_7b import hires_case, seeded_cache_rows, weights_7b  # noqa: E402


def gpu_forward(ctx, kv, tokens, P, embeds=None):
    B, L = tokens.shape
    logits = torch.empty(B, L, ctx.cfg.vocab, device=DEV)
    mulo.mulo_verify_forward(ctx, kv, B, L, P, dev(tokens), embeds, logits)
    torch.cuda.synchronize()
    return logits.cpu().numpy()


def cache_error(dec, kv, B, rows):
    """|device cache - oracle cache| over rows [0, rows), in the oracle's layout."""
    k = kv[0].float().cpu().permute(0, 1, 3, 2, 4)[:, :B, :rows]      # -> [nl, B, S, nh, dh]
    v = kv[1].float().cpu().permute(0, 1, 4, 2, 3)[:, :B, :rows]
    ek = (k.double() - dec.k[:, :B, :rows].double()).abs()
    ev = (v.double() - dec.v[:, :B, :rows].double()).abs()
    return ek, ev


def pair(m, w, cos, sin, B, S):
    return (OD.DecoderOracle(m, w, cos, sin, B, S, round_bf16=True),
            OD.DecoderOracle(m, w, cos, sin, B, S, round_bf16=False))


def test_forward_tiny_f32():
    c = WC.get("cfg1")
    m, B, L, Pn = c["model"], c["B"], c["L"], c["prefix"]
    w = G.make_weights(m, seed=0)
    ctx, cos, sin = make_ctx(m, w, B, c["max_seq"] + 8, L)
    kv = mulo.alloc_kv(ctx, DEV)
    dec = OD.DecoderOracle(m, w, cos, sin, B, c["max_seq"] + 8, round_bf16=False)
    prefix = G.uniform_tokens((B, Pn), m["vocab"], 0, tag=0)
    block = G.uniform_tokens((B, L), m["vocab"], 0, tag=1)
    for tag, toks, P in (("tiny prefill", prefix, 0), ("tiny block", block, Pn)):
        err = np.abs(gpu_forward(ctx, kv, toks, P) - dec.forward(toks, P).numpy()).max()
        say("  %s: max|err| %.3g (tol 1e-4)" % (tag, err))
        assert err <= 1e-4
    ek, ev = cache_error(dec, kv, B, Pn + L)
    assert ek.max() < 1e-5 and ev.max() < 1e-5
    assert kv[0][:, :, :, Pn + L:].abs().max() == 0 and kv[1][:, :, :, :, Pn + L:].abs().max() == 0
    # token-by-token passes give the block pass (causality), on the device
    kv2 = mulo.alloc_kv(ctx, DEV)
    gpu_forward(ctx, kv2, prefix, 0)
    seq = np.concatenate([gpu_forward(ctx, kv2, block[:, j:j + 1], Pn + j) for j in range(24)], axis=1)
    blk = gpu_forward(ctx, kv, block, Pn)
    assert np.abs(seq - blk[:, :24]).max() < 1e-4


@pytest.mark.parametrize("nh,dh,f,V,B,L,P", [
    (3, 4, 30, 20, 1, 1, 0),          # nothing a multiple of 16, rows of 30 floats not 16-byte aligned, one token
    (2, 18, 44, 68, 2, 17, 3),        # a head of 18: 16 + 2; two query tiles, the second one query deep
    (2, 64, 176, 128, 3, 33, 31),     # whole blocks of the head, keys ending on a tile edge
    (2, 128, 90, 64, 1, 16, 49),      # the widest head of the tiled attention
    (1, 136, 64, 64, 2, 5, 7),        # wider: one workgroup per query
    (2, 16, 1030, 1028, 2, 1024, 0),  # gate|up and lm-head on 32 x 32 tiles with ragged columns; down on 16 x 16 with a K of 1030
    (17, 18, 310, 308, 2, 512, 9),    # every projection on 32 x 32 tiles, K of 306 and 310 (rows not 16-byte aligned), ragged columns
    (5, 64, 320, 320, 2, 512, 7),     # the same with aligned rows
])
def test_forward_f32_shapes(nh, dh, f, V, B, L, P):
    """The float32 projections and attention at the edges of their tiles.  Bar: 1e-4 as for the tiny configuration
    (sums of at most 1030 float32 products of order 1: 1030 * 2^-24 = 6e-5)."""
    m = dict(n_layers=2, d_model=nh * dh, n_heads=nh, head_dim=dh, d_ffn=f, vocab=V, dtype="f32", rms_eps=1e-5)
    w = G.make_weights(m, seed=3, std=0.1)
    S = P + L + 3
    ctx, cos, sin = make_ctx(m, w, B, S, max(L, P, 1))
    kv = mulo.alloc_kv(ctx, DEV)
    kv[1].fill_(float("nan"))         # cache columns nobody has written must not reach the result
    dec = OD.DecoderOracle(m, w, cos, sin, B, S, round_bf16=False)
    if P:
        prefix = G.uniform_tokens((B, P), V, 0, tag=0)
        assert np.abs(gpu_forward(ctx, kv, prefix, 0) - dec.forward(prefix, 0).numpy()).max() <= 1e-4
    block = G.uniform_tokens((B, L), V, 0, tag=1)
    err = np.abs(gpu_forward(ctx, kv, block, P) - dec.forward(block, P).numpy()).max()
    say("  f32 %s: max|err| %.3g" % ((nh, dh, f, V, B, L, P), err))
    assert err <= 1e-4


@pytest.mark.parametrize("nh,dh,f", [(4, 64, 688), (3, 18, 203)])
def test_forward_f32_has_the_same_bits_alone_in_a_batch_and_token_by_token(nh, dh, f):
    """Every float32 sum is added in an order that its own length fixes: the logits and cache rows of a sequence are the same
    bits alone, in batches of up to 9 (up to 1.8 million outputs a projection, past every size at which it changes its
    tile) and one token at a time.  The widths of the tiny configuration, and rows that are not 16-byte aligned."""
    m = dict(n_layers=2, d_model=nh * dh, n_heads=nh, head_dim=dh, d_ffn=f, vocab=1024, dtype="f32", rms_eps=1e-5)
    B, L, P = 9, 200, 11
    ctx, cos, sin = make_ctx(m, G.make_weights(m, seed=5), B, 224, L)
    kv = mulo.alloc_kv(ctx, DEV)
    gpu_forward(ctx, kv, G.uniform_tokens((1, P), 1024, 5, tag=0), 0)
    for t in kv:
        t[:, 1:].copy_(t[:, :1].expand_as(t[:, 1:]))
    many = G.uniform_tokens((B, L), 1024, 5, tag=1)
    many[:] = np.where(np.arange(B)[:, None] % 4 == 0, many[:1], many)
    one = gpu_forward(ctx, kv, many[:1], P)[0]
    k1, v1 = kv[0][:, 0, :, P:P + L].clone(), kv[1][:, 0, :, :, P:P + L].clone()
    for n in (2, 3, 5, 9):
        z = gpu_forward(ctx, kv, many[:n], P)
        for b in range(0, n, 4):
            assert np.array_equal(z[b], one), (n, b)
            assert torch.equal(kv[0][:, b, :, P:P + L], k1) and torch.equal(kv[1][:, b, :, :, P:P + L], v1), (n, b)
    for j in range(40):
        assert np.array_equal(gpu_forward(ctx, kv, many[:1, j:j + 1], P + j)[0, 0], one[j]), j


@pytest.mark.parametrize("nh,dh", [(2, 16), (2, 18), (4, 64), (2, 128), (1, 136)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_forward_f32_keeps_non_finite_positions_behind_the_causal_mask(nh, dh, bad):
    """A position whose embedding is not finite leaves every position before it as it is, bit for bit, and reaches itself
    and every position after it, wherever it lies in a tile of 16 queries or keys."""
    d, L, P = nh * dh, 37, 5
    m = dict(n_layers=2, d_model=d, n_heads=nh, head_dim=dh, d_ffn=48, vocab=64, dtype="f32", rms_eps=1e-5)
    ctx, cos, sin = make_ctx(m, G.make_weights(m, seed=6, std=0.1), 1, 48, L)
    kv = mulo.alloc_kv(ctx, DEV)
    toks = np.zeros((1, L), np.int32)
    gpu_forward(ctx, kv, G.uniform_tokens((1, P), 64, 6, tag=0), 0)
    emb = torch.randn(1, L, d, generator=torch.Generator(device=DEV).manual_seed(dh), device=DEV)
    clean = gpu_forward(ctx, kv, toks, P, emb)[0]
    for j in (0, 1, 10, 11, 26, 27, 36):
        e = emb.clone()
        e[0, j, 3] = bad
        z = gpu_forward(ctx, kv, toks, P, e)[0]
        assert np.array_equal(z[:j], clean[:j]), j
        assert not np.isfinite(z[j:]).any(), j


@pytest.mark.parametrize("nh,dh", [(8, 128), (16, 64)])
def test_a_row_has_the_same_bits_in_every_block_of_more_than_128_queries(nh, dh):
    """The attention of a row adds its keys in one order whatever the length of the block and the number of sequences: the
    rows of a 200-query block (one sequence, and 17 of them: past one 128-query workgroup per CU) are those of blocks of
    129, 256, 257 and 520 queries that begin with the same tokens, bit for bit."""
    m = dict(n_layers=1, d_model=nh * dh, n_heads=nh, head_dim=dh, d_ffn=256, vocab=512, dtype="bf16", rms_eps=1e-5)
    w, P, B = G.make_weights(m, seed=9), 75, 17
    ctx, cos, sin = make_ctx(m, w, B, 600, 520)
    kv = mulo.alloc_kv(ctx, DEV)
    gpu_forward(ctx, kv, G.uniform_tokens((1, P), 512, 9, tag=0), 0)
    for t in kv:
        t[:, 1:].copy_(t[:, :1].expand_as(t[:, 1:]))
    blk = G.uniform_tokens((1, 520), 512, 9, tag=1)
    ref = gpu_forward(ctx, kv, blk, P)[0]
    for L in (129, 200, 256, 257, 520):
        assert np.array_equal(gpu_forward(ctx, kv, blk[:, :L], P)[0], ref[:L]), L
        many = np.repeat(blk[:, :L], B, axis=0)
        many[1:-1, 0] = G.uniform_tokens((B - 2,), 512, 9, tag=2)
        z = gpu_forward(ctx, kv, many, P)
        assert np.array_equal(z[0], ref[:L]) and np.array_equal(z[-1], ref[:L]), L


@pytest.mark.parametrize("d,nh,f,V", [
    (768, 6, 8256, 1092),    # gate | up on 64 x 128 and 128 x 256; K of 129 steps for down, a ragged last column tile for the lm-head
    (768, 6, 704, 16384),    # the lm-head on 128 x 128, 128 x 256 and 256 x 256; K of 11 steps
    (1024, 16, 2112, 1092),  # down on small tiles up to 128 x 64; K of 33 steps
    (128, 2, 192, 260),      # K of 2 and 3 steps, fewer than the ring has stages
])
def test_every_tile_gives_the_same_sums(d, nh, f, V):
    """The projections of a launch run on the tile its sizes ask for; every tile adds the same products in the same order.
    One sequence alone (161 tokens, checked against the oracle) and as the first and last of launches of up to 2576
    tokens (no count is a multiple of a tile): the same logits and cache rows, bit for bit.  Which tiles that comes to
    is the rule's choice; the test below runs each of them."""
    m = dict(n_layers=1, d_model=d, n_heads=nh, head_dim=d // nh, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    L, P, S, Bmax = 161, 5, 168, 16
    w = G.make_weights(m, seed=21)
    ctx, cos, sin = make_ctx(m, w, Bmax, S, 164)
    kv = mulo.alloc_kv(ctx, DEV)
    dr, du = pair(m, w, cos, sin, 1, S)
    pre, blk = G.uniform_tokens((1, P), V, 21, tag=0), G.uniform_tokens((1, L), V, 21, tag=1)
    for t in (dr, du):
        t.forward(pre, 0)
    gpu_forward(ctx, kv, pre, 0)
    for t in kv:                      # every sequence behind the same prefix rows (a prefix launch of its own would stream or not)
        t[:, 1:].copy_(t[:, :1].expand_as(t[:, 1:]))
    one = gpu_forward(ctx, kv, blk, P)
    check_bf16_logits("161 tokens alone, width %d" % d, one, dr.forward(blk, P).numpy(), du.forward(blk, P).numpy())
    k1, v1 = kv[0][0, 0, :, P:P + L].clone(), kv[1][0, 0, :, :, P:P + L].clone()
    for B in (2, 5, 8, 13, 16):
        many = G.uniform_tokens((B, L), V, 21, tag=2)
        many[0] = many[-1] = blk[0]
        z = gpu_forward(ctx, kv, many, P)
        for b in (0, B - 1):
            assert np.array_equal(z[b], one[0]), (B, b)
            assert torch.equal(kv[0][0, b, :, P:P + L], k1) and torch.equal(kv[1][0, b, :, :, P:P + L], v1), (B, b)


@pytest.mark.parametrize("d,nh,f,V,B", [
    (128, 2, 192, 260, (1, 5)),        # K of 2 steps (q|k|v, out, gate|up, lm-head) and 3 (down); ragged columns
    (256, 4, 320, 1280, (1, 5)),       # 4 and 5; the lm-head and q|k|v on whole 256 x 256 tiles
    (384, 3, 384, 516, (1, 5)),        # 6 and 6; half a tile of 256 columns for q|k|v, out and the lm-head
    (768, 6, 1152, 1536, (1, 5)),      # 12 and 18; every projection has 256 x 256 tiles
    (256, 2, 704, 6656, (16,)),        # 11 x 26 tiles of 256 x 256 for the lm-head: the last columns are cut off (128 x 256)
])
def test_every_projection_on_every_tile_it_has(d, nh, f, V, B):
    """Each of q|k|v, out, gate|up, down and lm-head on each tile of the table that it has, against the rule's choice (which
    the oracle checks for one sequence): the same logits, cache rows, bit for bit.  161 tokens a sequence: no launch is
    a whole number of row tiles.  The rings see K from shorter than their stages to several times as long, the paired one
    (128 x 128, five stages) every remainder of its loop: 2 to 6 steps."""
    m = dict(n_layers=1, d_model=d, n_heads=nh, head_dim=d // nh, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    L, P, S = 161, 5, 168
    w = G.make_weights(m, seed=23)
    ctx, cos, sin = make_ctx(m, w, max(B), S, 164)
    kv = mulo.alloc_kv(ctx, DEV)
    pre = G.uniform_tokens((1, P), V, 23, tag=0)
    gpu_forward(ctx, kv, pre, 0)
    for t in kv:
        t[:, 1:].copy_(t[:, :1].expand_as(t[:, 1:]))
    widths = (3 * d, d, 2 * f, d, V)
    for n in B:
        toks = G.uniform_tokens((n, L), V, 23, tag=1)
        base = gpu_forward(ctx, kv, toks, P)
        if n == 1:
            dr, du = pair(m, w, cos, sin, 1, S)
            for t in (dr, du):
                t.forward(pre, 0)
            check_bf16_logits("width %d" % d, base, dr.forward(toks, P).numpy(), du.forward(toks, P).numpy())
        k0, v0 = kv[0][:, :n, :, P:P + L].clone(), kv[1][:, :n, :, :, P:P + L].clone()
        for i, (bm, bn) in enumerate(TILES):
            tiles_of(ctx, i)
            kv[0][:, :, :, P:].fill_(float("nan"))
            kv[1][:, :, :, :, P:].fill_(float("nan"))
            z = gpu_forward(ctx, kv, toks, P)
            for p, t in enumerate(tiles_of(ctx, -1)):
                whole = widths[p] % 256 == 0 and (p != 0 or d % 256 == 0)
                has = (i not in (0, 1, 2) if p == 2 else i != 3) and (i != 7 or whole) and (p != 0 or d % bn == 0)
                assert t == i or not has, (p, i, t)
            assert np.array_equal(z, base), (n, i)
            assert torch.equal(kv[0][:, :n, :, P:P + L], k0) and torch.equal(kv[1][:, :n, :, :, P:P + L], v0), (n, i)


@pytest.mark.parametrize("d,nh,f,V,B,L", [
    (128, 2, 256, 25600, 5, 161),   # K of 2 steps; the lm-head's 400 tiles are two rounds, the second one partly filled
    (384, 3, 256, 25600, 5, 161),   # the same with K of 6 steps
    (256, 2, 192, 512, 5, 161),     # down: K of 3 steps, fewer than the ring is deep
    (256, 4, 192, 512, 13, 161),    # sequences of 161 tokens end inside runs of 8: every V run of them, heads of 64
    (256, 2, 256, 512, 90, 3),      # three sequences in a run of 8
    (512, 4, 640, 512, 41, 811),    # 130 row tiles: q|k|v 780 tiles, out 260, gate|up 650, down 260 (K of 10 steps), lm-head 260
    (512, 8, 192, 768, 41, 811),    # down: K of 3 steps over two rounds; the lm-head 390 tiles; heads of 64
])
def test_256_tiles_at_short_k_and_over_rounds(d, nh, f, V, B, L):
    """256 x 256 tiles against 128 x 128 ones where the loads of a workgroup's next tile begin in the first steps of the one
    before, and where the last tile of a workgroup has no next: the same logits and cache rows, bit for bit, whatever the
    parity of the cache row a block begins at.  In a launch of more tiles than CUs a workgroup goes from one to the next: from
    one rotary or V tile to the other kind, and from one residual tile's stores to the next one's requests."""
    m = dict(n_layers=1, d_model=d, n_heads=nh, head_dim=d // nh, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    S = (L + 22) // 8 * 8
    w = G.make_weights(m, seed=25)
    ctx, cos, sin = make_ctx(m, w, B, S, (L + 3) // 4 * 4)
    kv = mulo.alloc_kv(ctx, DEV)
    toks = G.uniform_tokens((B, L), V, 25, tag=1)
    for P in (8, 9, 12):
        got = []
        for i in (4, 7):
            tiles_of(ctx, i)
            for t in kv:
                t.fill_(0.25)
            z = gpu_forward(ctx, kv, toks, P)
            ran = tiles_of(ctx, -1)
            assert (i == 4) == (7 not in ran), ran
            got.append((z, kv[0].clone(), kv[1].clone()))
        assert np.array_equal(got[0][0], got[1][0]), P
        assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][2], got[1][2]), P


def test_256_tiles_with_scattered_slots():
    """An island pass of more slots than stream (13 of each of 23 sequences, two of them unused) on 256 x 256 tiles against
    128 x 128 ones: cache rows, logit rows and tokens, bit for bit, and nothing written for an unused slot."""
    d, nh, V, B, L, P, n = 256, 2, 512, 23, 160, 7, 13
    m = dict(n_layers=2, d_model=d, n_heads=nh, head_dim=d // nh, d_ffn=512, vocab=V, dtype="bf16", rms_eps=1e-5)
    w = G.make_weights(m, seed=27)
    ctx, cos, sin = make_ctx(m, w, B, 168, L)
    kv = mulo.alloc_kv(ctx, DEV)
    g = torch.Generator(device=DEV).manual_seed(27)
    for t in kv:
        t.normal_(generator=g)
    first = [t.clone() for t in kv]
    mask = torch.zeros(B, L, dtype=torch.uint8, device=DEV)
    mask[:, torch.arange(n - 2, device=DEV) * 14 + 3] = 1
    rank = mask.to(torch.int32) - 1
    toks = dev(G.uniform_tokens((B, L), V, 27, tag=1))
    prev = dev(G.uniform_tokens((B,), V, 27, tag=2))
    got = []
    for i in (4, 7):
        tiles_of(ctx, i)
        for t, t0 in zip(kv, first):
            t.copy_(t0)
        out, logits = toks.clone(), torch.zeros(B, L, V, device=DEV)
        mulo.mulo_resample_islands(ctx, kv, B, P, L, 1, n, 5, 3, prev, mask, rank, out, logits)
        torch.cuda.synchronize()
        assert (7 in tiles_of(ctx, -1)) == (i == 7)
        got.append((out, logits, kv[0].clone(), kv[1].clone()))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    untouched = mask == 0
    assert torch.equal(got[0][3][:, :, :, :, P:P + L].permute(0, 1, 4, 2, 3)[:, untouched], first[1][:, :, :, :, P:P + L].permute(0, 1, 4, 2, 3)[:, untouched])



def test_forward_small_bf16_chained_blocks():
    c = WC.get("cfg2")
    m, B, L, Pn = c["model"], c["B"], c["L"], c["prefix"]
    w = G.make_weights(m, seed=0)
    ctx, cos, sin = make_ctx(m, w, B, c["max_seq"], L)
    kv = mulo.alloc_kv(ctx, DEV)
    dr, du = pair(m, w, cos, sin, B, c["max_seq"])
    prefix = G.uniform_tokens((B, Pn), m["vocab"], 0, tag=0)
    check_bf16_logits("small prefill", gpu_forward(ctx, kv, prefix, 0), dr.forward(prefix, 0).numpy(),
                      du.forward(prefix, 0).numpy())
    P = Pn
    for blk in range(3):                                    # cache append at n0 = 0, 256, 512
        toks = G.uniform_tokens((B, L), m["vocab"], 0, tag=10 + blk)
        check_bf16_logits("small block %d (P=%d)" % (blk, P), gpu_forward(ctx, kv, toks, P),
                          dr.forward(toks, P).numpy(), du.forward(toks, P).numpy())
        P += L
    ek, ev = cache_error(dr, kv, B, P)
    # layer 0 sees identical inputs on both sides: its cache rows agree up to rare one-ulp bf16 flips
    # (a flipped input element moves every output of its row by a little, hence the absolute part)
    tol_k = 2.0 ** -6 * (dr.k[0, :B, :P].double().abs() + 0.1)
    tol_v = 2.0 ** -6 * (dr.v[0, :B, :P].double().abs() + 0.1)
    say("  layer-0 cache: K mismatching %.4f%% (max %.3g, beyond tol %d)  V mismatching %.4f%% (max %.3g, beyond tol %d)" % (
        100 * (ek[0] > 0).double().mean(), ek[0].max(), int((ek[0] > tol_k).sum()),
        100 * (ev[0] > 0).double().mean(), ev[0].max(), int((ev[0] > tol_v).sum())))
    for name, e_, t_ in (("K", ek[0], tol_k), ("V", ev[0], tol_v)):
        bad = (e_ > t_).nonzero()
        if len(bad):
            say("  %s violations at [b, row, head, c]: %r" % (name, bad[:8].tolist()))
    assert (ek[0] <= tol_k).all() and (ev[0] <= tol_v).all()
    assert (ek[0] > 0).double().mean() < 0.01 and (ev[0] > 0).double().mean() < 0.01
    # deeper layers drift with the format's noise but stay close
    assert ek.max() < 0.25 and ev.max() < 0.25


def test_forward_single_layer_bf16():
    """One decoder layer + lm-head at the small and at the 7B-class width.  At
    the small width the stated 2e-2 holds; at the 7B width one layer's own
    rounding noise already exceeds it (logit std 1.28)."""
    for name, L, P in (("small", 256, 64), ("7b", 192, 64)):
        m = dict(WC.model(name), n_layers=1)
        w = G.make_weights(m, seed=3)
        S = P + L
        ctx, cos, sin = make_ctx(m, w, 2, S, L)
        kv = mulo.alloc_kv(ctx, DEV)
        dr, du = pair(m, w, cos, sin, 2, S)
        pre = G.uniform_tokens((2, P), m["vocab"], 3, tag=0)
        blk = G.uniform_tokens((2, L), m["vocab"], 3, tag=1)
        gpu_forward(ctx, kv, pre, 0)
        dr.forward(pre, 0)
        du.forward(pre, 0)
        check_bf16_logits("1-layer %s" % name, gpu_forward(ctx, kv, blk, P), dr.forward(blk, P).numpy(),
                          du.forward(blk, P).numpy(), strict=(name == "small"))


def test_forward_ragged_shapes_bf16():
    # M = 300 (not a tile multiple), vocabulary 1000 (ragged last column tile), odd prefix length
    m = dict(n_layers=2, d_model=256, n_heads=4, head_dim=64, d_ffn=320, vocab=1000, dtype="bf16", rms_eps=1e-5)
    B, L, Pn, S = 3, 100, 37, 144
    w = G.make_weights(m, seed=5, std=0.05)
    ctx, cos, sin = make_ctx(m, w, B, S, L)
    kv = mulo.alloc_kv(ctx, DEV, zero=False)
    kv[0].fill_(float("nan"))                               # rows not yet written must never be used
    kv[1].fill_(float("nan"))
    dr, du = pair(m, w, cos, sin, B, S)
    prefix = G.uniform_tokens((B, Pn), m["vocab"], 5, tag=0)
    block = G.uniform_tokens((B, L), m["vocab"], 5, tag=1)
    check_bf16_logits("ragged prefill", gpu_forward(ctx, kv, prefix, 0), dr.forward(prefix, 0).numpy(),
                      du.forward(prefix, 0).numpy())
    check_bf16_logits("ragged block", gpu_forward(ctx, kv, block, Pn), dr.forward(block, Pn).numpy(),
                      du.forward(block, Pn).numpy())
    # head_dim 128 variant with a single short block
    m2 = dict(n_layers=1, d_model=256, n_heads=2, head_dim=128, d_ffn=192, vocab=512, dtype="bf16", rms_eps=1e-5)
    w2 = G.make_weights(m2, seed=6, std=0.05)
    ctx2, cos2, sin2 = make_ctx(m2, w2, 2, 80, 72)
    kv2 = mulo.alloc_kv(ctx2, DEV)
    d2r, d2u = pair(m2, w2, cos2, sin2, 2, 80)
    t2 = G.uniform_tokens((2, 72), 512, 6)
    check_bf16_logits("dh128 block", gpu_forward(ctx2, kv2, t2, 0), d2r.forward(t2, 0).numpy(),
                      d2u.forward(t2, 0).numpy())


def test_forward_embeds_input_and_errors():
    m = dict(n_layers=1, d_model=128, n_heads=2, head_dim=64, d_ffn=128, vocab=256, dtype="bf16", rms_eps=1e-5)
    w = G.make_weights(m, seed=7, std=0.05)
    ctx, cos, sin = make_ctx(m, w, 2, 64, 32)
    kv = mulo.alloc_kv(ctx, DEV)
    toks = G.uniform_tokens((2, 32), 256, 7)
    a = gpu_forward(ctx, kv, toks, 0)
    emb = w["embed"][torch.as_tensor(toks).long()].to(DEV).contiguous()
    b = gpu_forward(ctx, kv, toks * 0, 0, embeds=emb)
    assert np.array_equal(a, b)
    for bad in [dict(B=3, L=32, P=0), dict(B=2, L=40, P=0), dict(B=2, L=32, P=40)]:
        with pytest.raises(mulo.MuloError) as e:
            mulo.mulo_verify_forward(ctx, kv, bad["B"], bad["L"], bad["P"], torch.zeros(3, 40, dtype=torch.int32, device=DEV),
                                     None, torch.empty(3, 40, 256, device=DEV))
        assert e.value.status == 2


@pytest.mark.parametrize("nh,dh,f,dtype", [(2, 64, 128, "bf16"), (9, 128, 256, "bf16"), (4, 64, 688, "f32"), (3, 18, 203, "f32")])
def test_embeddings_may_start_at_any_element(nh, dh, f, dtype):
    """Rows that allow 16-byte accesses and rows that do not (a start off by one element, a width of 54) are the same copy:
    one row, and several, given as tokens, as aligned embeddings and as unaligned ones have the same bits."""
    m = dict(n_layers=1, d_model=nh * dh, n_heads=nh, head_dim=dh, d_ffn=f, vocab=256, dtype=dtype, rms_eps=1e-5)
    w = G.make_weights(m, seed=9, std=0.05)
    ctx, cos, sin = make_ctx(m, w, 2, 64, 32)
    kv = mulo.alloc_kv(ctx, DEV)
    for B, L in ((1, 1), (2, 31)):
        toks = G.uniform_tokens((B, L), 256, 9)
        want = gpu_forward(ctx, kv, toks, 0)
        rows = w["embed"][torch.as_tensor(toks).long()].to(DEV).contiguous()
        off = torch.empty(rows.numel() + 1, dtype=rows.dtype, device=DEV)[1:].view(rows.shape).copy_(rows)
        assert rows.data_ptr() % 16 == 0 and off.data_ptr() % 16 != 0
        for e in (rows, off):
            assert np.array_equal(gpu_forward(ctx, kv, toks * 0, 0, embeds=e), want), (B, L)


@pytest.mark.timeout(900)
def test_forward_7b_first_block_and_teacher_forced_layers():
    """7B-class decoder, batch 1: real prefill of the 128-token prefix, then the
    first 576-token block (M = 576 is not a multiple of the 128/256 tiles); then
    layers 0, 15 and 31 alone, each fed the oracle's hidden state entering it."""
    c = WC.get("cfg3")
    m, B, L, Pn = c["model"], c["B"], c["L"], c["prefix"]
    w = weights_7b()
    ctx, cos, sin = make_ctx(m, w, B, c["max_seq"], L)
    kv = mulo.alloc_kv(ctx, DEV)
    dr, du = pair(m, w, cos, sin, B, Pn + L)
    prefix = G.uniform_tokens((B, Pn), m["vocab"], 0, tag=0)
    block = G.uniform_tokens((B, L), m["vocab"], 0, tag=1)
    say("7B prefill (oracle, rounded + exact) ...")
    check_bf16_logits("7B prefill", gpu_forward(ctx, kv, prefix, 0), dr.forward(prefix, 0).numpy(),
                      du.forward(prefix, 0).numpy())
    say("7B block (oracle, rounded + exact) ...")
    taps = []
    zr = dr.forward(block, Pn, taps=taps).numpy()
    check_bf16_logits("7B block", gpu_forward(ctx, kv, block, Pn), zr, du.forward(block, Pn).numpy())
    del ctx, kv
    wd = device_weights(w)
    m1 = dict(m, n_layers=1)
    for l in (0, 15, 31):
        sl = lambda t: t[l:l + 1] if t.dim() == 3 or (t.dim() == 2 and t.shape[0] == m["n_layers"]) else t
        w1 = {k: sl(v) for k, v in w.items()}
        wd1 = {k: sl(v) for k, v in wd.items()}
        x_in = taps[l].to(torch.bfloat16)                       # hidden state entering layer l, as the bf16 input
        ctx1, cos1, sin1 = make_ctx_from_device(m1, wd1, B, L, L)
        kv1 = mulo.alloc_kv(ctx1, DEV)
        d1r, d1u = pair(m1, w1, cos1, sin1, B, L)
        zg = gpu_forward(ctx1, kv1, block * 0, 0, embeds=x_in.to(DEV).contiguous())
        emb = x_in.double().numpy()
        check_bf16_logits("7B layer %d teacher-forced" % l, zg, d1r.forward(block * 0, 0, embeds=emb).numpy(),
                          d1u.forward(block * 0, 0, embeds=emb).numpy())
        del ctx1, kv1


def fill_device_cache(kv, m, P, B):
    """Seeded N(0, 1) rows [0, P) of every batch element, as tests.cases_7b.seeded_cache_rows makes them."""
    for b in range(B):
        kb, vb = seeded_cache_rows(m, P, b)                                  # [nl, nh, P, dh]
        kv[0][:, b, :, :P] = kb.to(DEV)
        kv[1][:, b, :, :, :P] = vb.permute(0, 1, 3, 2).to(DEV)


@pytest.mark.timeout(900)
def test_forward_7b_hires_full_launch_sampled_sequence():
    """Config-4 launch (B = 4, L = 1024, P = 3200: the largest cache) on the
    device; the oracle recomputes batch element 0 in full.  Cache rows [0, P) are
    seeded N(0, 1) values on both sides (a real prefill of 3200 rows is hours of
    CPU time); the inputs are the sigma recipe's provisional up-sampled draft."""
    h = hires_case()
    c, P, toks = h["c"], h["P"], h["inp"]
    m, B, L = c["model"], c["B"], c["L"]
    w = weights_7b()
    ctx, cos, sin = make_ctx(m, w, B, c["max_seq"], L)
    kv = mulo.alloc_kv(ctx, DEV)
    fill_device_cache(kv, m, P, B)
    zg = gpu_forward(ctx, kv, toks, P)
    check_bf16_logits("7B hi-res b=0", zg[:1], h["z_r"], h["z_u"])
    say("  logits above 2e-2 of the oracle's: %d of %d" % (int((np.abs(zg[:1] - h["z_r"]) > 2e-2).sum()), h["z_r"].size))
    # batch elements are independent: element 3 alone reproduces its rows of the batched launch
    kv1 = (kv[0][:, 3:4].contiguous(), kv[1][:, 3:4].contiguous())
    ctx1, _, _ = make_ctx(m, w, 1, c["max_seq"], L)
    z3 = gpu_forward(ctx1, kv1, toks[3:4], P)
    say("  batch element 3 alone vs in the batch: max diff %.3g" % np.abs(z3 - zg[3:4]).max())
    assert np.abs(z3 - zg[3:4]).max() <= 1e-3
    del ctx, ctx1


@pytest.mark.parametrize("dh,nh,copy", [(64, 4, False), (128, 2, False), (128, 2, True)])
def test_forward_single_token_steps_with_split_keys(dh, nh, copy):
    """Decode shape: one token per sequence against a cache of several key tiles, so that the keys are dealt
    to several workgroups per head and combined (and the projections run in the weight-streaming kernel).
    Cache lengths 199 .. 202 straddle a tile boundary (64-key tiles, the last one partly filled)."""
    m = dict(n_layers=2, d_model=dh * nh, n_heads=nh, head_dim=dh, d_ffn=512, vocab=1024, dtype="bf16", rms_eps=1e-5)
    B, Pn = 3, 199
    w = G.make_weights(m, seed=5)
    ctx, cos, sin = make_ctx(m, w, B, 208, 200, stream_copy=copy)   # copy: the weights once more in fragment order
    kv = mulo.alloc_kv(ctx, DEV)
    dr, du = pair(m, w, cos, sin, B, 208)
    pre = G.uniform_tokens((B, Pn), m["vocab"], 5, tag=0)
    gpu_forward(ctx, kv, pre, 0)
    dr.forward(pre, 0)
    du.forward(pre, 0)
    for step in range(4):
        t = G.uniform_tokens((B, 1), m["vocab"], 5, tag=10 + step)
        check_bf16_logits("single token, %d cached rows, dh %d" % (Pn + step, dh), gpu_forward(ctx, kv, t, Pn + step),
                          dr.forward(t, Pn + step).numpy(), du.forward(t, Pn + step).numpy(), strict=True)


@pytest.mark.parametrize("dh,nh", [(64, 4), (128, 2)])
@pytest.mark.parametrize("L,P,S", [
    (1, 71, 72),       # a token whose cache ends 8 rows into a 64-key tile (keys dealt to several workgroups)
    (7, 113, 120),     # and 56 rows into one
    (100, 92, 192),    # whole tiles
    (128, 128, 264),   # 8 free rows behind the block
    (130, 134, 264),   # 128-key tiles: 8 rows into the last one
    (300, 204, 504),   # 120 rows into it
])
def test_attention_at_the_end_of_the_cache(dh, nh, L, P, S):
    """A cache that ends inside a tile of keys against one with 128 more rows, NaN in every row that nothing has written: the same
    logits and cache rows, bit for bit."""
    m = dict(n_layers=2, d_model=dh * nh, n_heads=nh, head_dim=dh, d_ffn=256, vocab=512, dtype="bf16", rms_eps=1e-5)
    B = 2
    w = G.make_weights(m, seed=29)
    toks = G.uniform_tokens((B, L), m["vocab"], 29, tag=1)
    g = torch.Generator(device=DEV).manual_seed(29)
    k0 = torch.randn(2, B, nh, P, dh, generator=g, device=DEV)
    v0 = torch.randn(2, B, nh, dh, P, generator=g, device=DEV)
    got = []
    for rows in (S, S + 128):
        ctx, cos, sin = make_ctx(m, w, B, rows, (L + 3) // 4 * 4)
        kv = mulo.alloc_kv(ctx, DEV)
        for t in kv:
            t.fill_(float("nan"))
        kv[0][:, :, :, :P] = k0
        kv[1][:, :, :, :, :P] = v0
        z = gpu_forward(ctx, kv, toks, P)
        assert np.isfinite(z).all()
        got.append((z, kv[0][:, :, :, :P + L].clone(), kv[1][:, :, :, :, :P + L].clone()))
    assert np.array_equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][2], got[1][2])


def frag_to_rows(buf, M, K):
    """Undo the fragment order of a [M, K] token operand (include/mulo.h, mulo_workspace_read): element (m, k)
    sits at ((m / 16) * (K / 32) + k / 32) * 512 + ((k % 32) / 8 * 16 + m % 16) * 8 + k % 8."""
    m = np.arange(M)[:, None]
    k = np.arange(K)[None, :]
    idx = ((m // 16) * (K // 32) + k // 32) * 512 + ((k % 32) // 8 * 16 + m % 16) * 8 + k % 8
    return buf.reshape(-1)[idx]


@pytest.mark.parametrize("B,L,copy", [(3, 1, False), (4, 13, False), (2, 32, False), (3, 1, True), (4, 13, True),
                                      (4, 40, True), (2, 100, True), (2, 95, True), (3, 79, True), (4, 64, True)])
def test_forward_few_tokens_keeps_its_operands_in_fragment_order(B, L, copy):
    """Launches of at most 64 tokens (one, four and four token groups of 16; 3, 52 and 64 tokens) run every projection
    in the weight-streaming kernel, whose token operand the producing kernels leave in the matrix instruction's own
    order; with the context's weight copy in fragment order so do launches of up to 256 tokens (160 to 256 here, 10 to 16 groups: the
    kernel that shares the token operand through LDS and deals K to several workgroups).  One layer: the attention output and silu(gate) * up read back through mulo_workspace_read, put back in
    row order by the documented formula, are the oracle's stage tensors; the logits are held to the usual bound."""
    m = dict(n_layers=1, d_model=256, n_heads=2, head_dim=128, d_ffn=512, vocab=1024, dtype="bf16", rms_eps=1e-5)
    Pn, S, M = 70, 184, B * L
    w = G.make_weights(m, seed=11)
    ctx, cos, sin = make_ctx(m, w, B, S, 104, stream_copy=copy)
    kv = mulo.alloc_kv(ctx, DEV)
    dr, du = pair(m, w, cos, sin, B, S)
    pre = G.uniform_tokens((B, Pn), m["vocab"], 11, tag=0)
    gpu_forward(ctx, kv, pre, 0)
    dr.forward(pre, 0)
    du.forward(pre, 0)
    blk = G.uniform_tokens((B, L), m["vocab"], 11, tag=1)
    stages = {}
    z_r = dr.forward(blk, Pn, stages=stages).numpy()
    z = gpu_forward(ctx, kv, blk, Pn)
    check_bf16_logits("%d x %d tokens, weight-streaming projections" % (B, L), z, z_r, du.forward(blk, Pn).numpy(), strict=True)
    M16 = (M + 15) // 16 * 16
    for name, which, K in (("att", mulo.MULO_WS_ATTN, m["d_model"]), ("hmid", mulo.MULO_WS_FFN, m["d_ffn"])):
        buf = torch.empty(M16 * K, dtype=torch.bfloat16, device=DEV)
        mulo.mulo_workspace_read(ctx, which, buf)
        torch.cuda.synchronize()
        got = frag_to_rows(buf.float().cpu().numpy(), M, K)
        want = stages[name][0].reshape(M, K).double().numpy()
        err = np.abs(got - want)
        tol = 2.0 ** -5 * (np.abs(want) + np.sqrt((want ** 2).mean()))
        say("  %s in fragment order, %d tokens: max|err| %.3g, beyond tolerance %d of %d" % (name, M, err.max(), (err > tol).sum(), err.size))
        assert (err > tol).mean() <= 0.005 and err.max() <= 0.25 * np.abs(want).max()


@pytest.mark.parametrize("d,nh,f,V", [
    (1408, 11, 4160, 12308),   # q|k|v 264 blocks of 16 columns: two a workgroup; gate|up 260 (halves for one token group); lm-head 770, a ragged last one
    (768, 6, 8256, 16388),     # gate|up 516 blocks: two and three; lm-head 1025: a workgroup's last blocks lie past the end; down: 258 steps in 8 slices
])
def test_streamed_sums_do_not_depend_on_the_columns_a_workgroup_takes(d, nh, f, V):
    """Blocks of 5 to 64 tokens (one to four token groups: other column blocks per workgroup; from two groups on, K of 4096 and more in
    slices that the norm adds), with the weight copy and without: the rows they share are the same bits, those of 64 tokens are the
    oracle's."""
    m = dict(n_layers=1, d_model=d, n_heads=nh, head_dim=d // nh, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    w, P, S = G.make_weights(m, seed=31), 9, 80
    pre, blk = G.uniform_tokens((1, P), V, 31, tag=0), G.uniform_tokens((1, 64), V, 31, tag=1)
    ref = None
    for copy in (False, True):
        ctx, cos, sin = make_ctx(m, w, 1, S, 64, stream_copy=copy)
        kv = mulo.alloc_kv(ctx, DEV)
        gpu_forward(ctx, kv, pre, 0)
        for L in (64, 48, 40, 32, 17, 16, 5):
            z = gpu_forward(ctx, kv, blk[:, :L], P)
            if ref is None:
                dr, du = pair(m, w, cos, sin, 1, S)
                for t in (dr, du):
                    t.forward(pre, 0)
                zr, zu = dr.forward(blk, P).numpy(), du.forward(blk, P).numpy()
                check_bf16_logits("64 streamed tokens, width %d" % d, z, zr, zu)
                ref = z
                k1, v1 = kv[0][0, 0, :, P:P + 64].clone(), kv[1][0, 0, :, :, P:P + 64].clone()
            assert np.array_equal(z, ref[:, :L]), (copy, L)
            assert torch.equal(kv[0][0, 0, :, P:P + L], k1[:, :L]) and torch.equal(kv[1][0, 0, :, :, P:P + L], v1[:, :, :L]), (copy, L)


@pytest.mark.parametrize("L", [65, 128, 129, 192])
def test_a_few_hundred_tokens_with_long_residual_projections(L):
    """65 to 192 tokens, out and down of 3072 x 3072 and 3072 x 4160: logits, residual stream and cache rows against the oracle, and
    against the same rows of a launch of 193 tokens: the same bits from 129 tokens on (up to 128 the attention adds its keys over
    other tiles)."""
    nh, dh, f, V = 24, 128, 4160, 12 * 1024
    m = dict(n_layers=1, d_model=nh * dh, n_heads=nh, head_dim=dh, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    w, P, S = G.make_weights(m, seed=33), 5, 200
    ctx, cos, sin = make_ctx(m, w, 1, S, 196)
    kv = mulo.alloc_kv(ctx, DEV)
    pre, blk = G.uniform_tokens((1, P), V, 33, tag=0), G.uniform_tokens((1, 193), V, 33, tag=1)
    gpu_forward(ctx, kv, pre, 0)
    whole = gpu_forward(ctx, kv, blk, P)
    assert min(tiles_of(ctx, -1)) >= 0
    k1, v1 = kv[0][0, 0, :, P:P + L].clone(), kv[1][0, 0, :, :, P:P + L].clone()
    x = torch.empty(193, nh * dh, device=DEV)
    mulo.mulo_workspace_read(ctx, mulo.MULO_WS_RESIDUAL, x)
    z = gpu_forward(ctx, kv, blk[:, :L], P)
    xs = torch.empty(L, nh * dh, device=DEV)
    mulo.mulo_workspace_read(ctx, mulo.MULO_WS_RESIDUAL, xs)
    torch.cuda.synchronize()
    dr, du = pair(m, w, cos, sin, 1, S)
    for t in (dr, du):
        t.forward(pre, 0)
    check_bf16_logits("%d tokens" % L, z, dr.forward(blk[:, :L], P).numpy(), du.forward(blk[:, :L], P).numpy())
    assert torch.equal(kv[0][0, 0, :, P:P + L], k1) and torch.equal(kv[1][0, 0, :, :, P:P + L], v1)
    if L > 128:
        assert torch.equal(xs, x[:L]) and np.array_equal(z, whole[:, :L])
    # up to 128 tokens the attention's sums differ in float32, and by what bf16 roundings make of that (a flipped one moves a row's
    # products by 2^-8 of one term): 2^-7 of a residual's size bounds both
    err = (xs - x[:L]).abs().max() / x[:L].abs().max()
    say("  residual stream against 193 tokens: %.3g of the largest" % float(err))
    assert float(err) <= 2.0 ** -7 and np.abs(z - whole[:, :L]).max() <= 2.0 ** -5 * np.abs(whole).max()


_RANDOM_WEIGHTS = {}


def _random_device_weights(m):
    """Weights N(0, 0.02) made on the device, norms of gain 1."""
    key = tuple(sorted((k, str(v)) for k, v in m.items()))
    if key not in _RANDOM_WEIGHTS:
        _RANDOM_WEIGHTS.clear()
        nl, d, f, V = m["n_layers"], m["d_model"], m["d_ffn"], m["vocab"]
        g = torch.Generator(device=DEV).manual_seed(1)
        shapes = dict(embed=(V, d), wq=(nl, d, d), wk=(nl, d, d), wv=(nl, d, d), wo=(nl, d, d), w_gate=(nl, f, d), w_up=(nl, f, d),
                      w_down=(nl, d, f), lm_head=(V, d))
        w = {k: torch.empty(s, dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g) for k, s in shapes.items()}
        w.update({k: torch.ones(s, dtype=torch.bfloat16, device=DEV) for k, s in (("attn_norm", (nl, d)), ("ffn_norm", (nl, d)), ("final_norm", (d,)))})
        _RANDOM_WEIGHTS[key] = w
    return _RANDOM_WEIGHTS[key]


def _same_bits_alone_and_in_batches(m, w, L, batches, P=8, copy=False, blocks=(256,)):
    """Sequence 0's logits, residual stream and cache rows in launches of `batches` sequences, in a context for each of `blocks`: the
    same bits."""
    nh, dh, d = m["n_heads"], m["head_dim"], m["d_model"]
    g = torch.Generator(device=DEV).manual_seed(L)
    pre = [torch.randn(m["n_layers"], 1, *s, generator=g, device=DEV).to(torch.bfloat16) for s in ((nh, P, dh), (nh, dh, P))]
    toks = G.uniform_tokens((max(batches), L), m["vocab"], 41, tag=L)
    ref = None
    for block in blocks:
        for B in batches if block == blocks[-1] else batches[:1]:
            ctx, _, _ = make_ctx_from_device(m, w, B if block < blocks[-1] else max(batches), 264, block, stream_copy=copy)
            kv = mulo.alloc_kv(ctx, DEV)
            kv[0][:, :, :, :P], kv[1][:, :, :, :, :P] = pre
            z = gpu_forward(ctx, kv, toks[:B], P)
            x = torch.empty(B * L, d, device=DEV)
            mulo.mulo_workspace_read(ctx, mulo.MULO_WS_RESIDUAL, x)
            torch.cuda.synchronize()
            got = (torch.tensor(z[0]), x[:L].clone(), kv[0][:, 0, :, P:P + L].clone(), kv[1][:, 0, :, :, P:P + L].clone())
            ref = ref or got
            for name, a, b in zip(("logits", "residual stream", "keys", "values"), got, ref):
                assert torch.equal(a, b), (name, B, block)


@pytest.mark.parametrize("L,batches", [(65, (1, 2, 3)), (96, (1, 2, 3)), (128, (1, 2)), (161, (1, 2)), (192, (1, 2))])
def test_wide_projections_have_the_same_bits_alone_and_in_a_batch(L, batches):
    """Width 4096, 4160 feed-forward columns, two layers (the second one's cache rows see the first one's out and down): a block of 65 to
    192 tokens alone and as the first of two or three sequences (130 to 384 tokens) adds every sum in the same order."""
    d, nh, f, V = 4096, 32, 4160, 16384
    m = dict(n_layers=2, d_model=d, n_heads=nh, head_dim=128, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    _same_bits_alone_and_in_batches(m, _random_device_weights(m), L, batches)


@pytest.mark.parametrize("L,batches", [(65, (1, 2, 3)), (100, (1, 2)), (128, (1, 2))])
@pytest.mark.parametrize("d,nh,f,V", [(1408, 11, 4160, 12308), (768, 6, 8256, 16388)])
def test_streamed_blocks_have_the_same_bits_alone_in_a_batch_and_in_any_context(d, nh, f, V, L, batches):
    """65 to 256 tokens with the weight copy, out and down in up to eight K slices that the norm adds: the deal is the projection's
    alone, so a block gets the same bits alone, in a batch of up to 256 tokens, and in a context that holds nothing but the block
    (the smallest scratch).  The lm-heads end inside a group of 128 columns."""
    m = dict(n_layers=2, d_model=d, n_heads=nh, head_dim=d // nh, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    _same_bits_alone_and_in_batches(m, _random_device_weights(m), L, batches, copy=True, blocks=((L + 3) // 4 * 4, 256))


@pytest.mark.parametrize("L", [65, 81, 128, 145, 160, 161, 256])
def test_streamed_blocks_of_a_few_hundred_tokens_against_the_oracle(L):
    """The same model and weight copy: five to sixteen token groups, the last one ragged or whole, down (4160 products, eight slices, the last
    one shorter) added by the final norm, against the oracle."""
    d, nh, f, V = 1408, 11, 4160, 12308
    m = dict(n_layers=1, d_model=d, n_heads=nh, head_dim=d // nh, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    w, P, S = G.make_weights(m, seed=35), 9, 272
    ctx, cos, sin = make_ctx(m, w, 1, S, 256, stream_copy=True)
    kv = mulo.alloc_kv(ctx, DEV)
    pre, blk = G.uniform_tokens((1, P), V, 35, tag=0), G.uniform_tokens((1, L), V, 35, tag=1)
    gpu_forward(ctx, kv, pre, 0)
    dr, du = pair(m, w, cos, sin, 1, S)
    for t in (dr, du):
        t.forward(pre, 0)
    check_bf16_logits("%d streamed tokens" % L, gpu_forward(ctx, kv, blk, P), dr.forward(blk, P).numpy(), du.forward(blk, P).numpy())


@pytest.mark.parametrize("d,nh,f", [(1024, 8, 4096), (1408, 11, 4160), (3072, 24, 4096)])
@pytest.mark.parametrize("copy", [False, True])
def test_a_norm_gives_the_same_bits_with_slices_to_add_and_without(d, nh, f, copy):
    """Weights of zero for down: whatever its K slices, they add nothing, so the norm behind it sees the same residual stream in every
    launch.  Four sequences of 16 tokens together (64 tokens: several slices from 4096 products on) and each alone (16: none): the
    same logits, bit for bit.  A scale that differs in its last bit shows in one bf16 value of 2^15 or fewer: 1024 rows, three norms
    each.  (The embedding's own values are of 8 bits, whose squares are exact: out adds the others.)"""
    V = 512
    m = dict(n_layers=3, d_model=d, n_heads=nh, head_dim=d // nh, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    w = dict(_random_device_weights(m))
    w["w_down"] = torch.zeros_like(w["w_down"])
    ctx, _, _ = make_ctx_from_device(m, w, 4, 16, 16, stream_copy=copy)
    kv = mulo.alloc_kv(ctx, DEV)
    for seed in range(16):
        emb = torch.randn(4, 16, d, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV).to(torch.bfloat16)
        z = gpu_forward(ctx, kv, np.zeros((4, 16), np.int32), 0, emb)
        for b in range(4):
            assert np.array_equal(gpu_forward(ctx, kv, np.zeros((1, 16), np.int32), 0, emb[b:b + 1].contiguous())[0], z[b]), (seed, b)


@pytest.mark.parametrize("d,nh,f", [(4096, 32, 4096), (2048, 16, 8192), (4224, 33, 4160), (8320, 65, 4096)])
@pytest.mark.parametrize("copy", [False, True])
def test_a_row_has_the_same_bits_in_every_streamed_block(d, nh, f, copy):
    """Out and down in slices in workgroups of 128 columns (the copy of widths that fill the chip) and of 64, one slice shorter than the
    others or as long, the norm over up to eight 16-byte pieces a thread and over longer rows: four sequences of 16 tokens
    together, three, two and each alone (no slices).  The logits and the cache rows of two layers, bit for bit."""
    V = 1024
    m = dict(n_layers=2, d_model=d, n_heads=nh, head_dim=d // nh, d_ffn=f, vocab=V, dtype="bf16", rms_eps=1e-5)
    ctx, _, _ = make_ctx_from_device(m, _random_device_weights(m), 4, 32, 16, stream_copy=copy)
    kv = mulo.alloc_kv(ctx, DEV)
    toks = G.uniform_tokens((4, 16), V, 43, tag=d)
    z = gpu_forward(ctx, kv, toks, 0)
    k4, v4 = kv[0].clone(), kv[1].clone()
    for B in (3, 2):
        assert np.array_equal(gpu_forward(ctx, kv, toks[:B], 0), z[:B]), B
        assert torch.equal(kv[0][:, :B, :, :16], k4[:, :B, :, :16]) and torch.equal(kv[1][:, :B, :, :, :16], v4[:, :B, :, :, :16]), B
    for b in range(4):
        assert np.array_equal(gpu_forward(ctx, kv, toks[b:b + 1], 0)[0], z[b]), b
        assert torch.equal(kv[0][:, 0, :, :16], k4[:, b, :, :16]) and torch.equal(kv[1][:, 0, :, :, :16], v4[:, b, :, :, :16]), b


def test_keys_have_the_same_bits_in_every_streamed_block():
    """The rotation of a pair rounds one of its products before it adds the other: which one must not follow the kernel.  It shows in one
    bf16 key of 2^16 or so: 1024 rows of 4096 channels, in blocks of one to four token groups, with the weight copy and without."""
    d, V = 4096, 512
    m = dict(n_layers=1, d_model=d, n_heads=32, head_dim=128, d_ffn=128, vocab=V, dtype="bf16", rms_eps=1e-5)
    w = _random_device_weights(m)
    for seed in range(16):
        emb = torch.randn(4, 16, d, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV).to(torch.bfloat16)
        ref = None
        for copy in (False, True):
            ctx, _, _ = make_ctx_from_device(m, w, 4, 16, 16, stream_copy=copy)
            kv = mulo.alloc_kv(ctx, DEV)
            for B in (1, 2, 3, 4):
                gpu_forward(ctx, kv, np.zeros((B, 16), np.int32), 0, emb[:B].contiguous())
                ref = kv[0][:, :1].clone() if ref is None else ref
                assert torch.equal(kv[0][:, :1], ref), (seed, copy, B)
