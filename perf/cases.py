"""The work that is timed: what a user of libmulo has it do, through the entry points of the binding.

Five kinds of case, each with the sizes of this repository's workloads (`workloads/configs.py`, `bench.py`):

  step     mulo_verify_step of the float32 model: up-sampling, target pass, accept test, expansion and re-draw.
  forward  mulo_verify_forward of a bf16 model: a drafted block against the cache (verification), a prefix from the
           embeddings (prefill), one token per sequence (sequential re-sampling, decoding).
  islands  mulo_resample_islands of a bf16 model: one pass over scattered single-position islands, which is what
           re-sampling comes to when only the rejected positions themselves are marked.
  decide   mulo_upsample_draft and mulo_accept_local_resample on given logits: the decision stage with Eq. 1 and the
           residual draw.
  guided   mulo_accept_local_resample with guidance, neighbour pooling and the threshold rule, then
           mulo_rejection_islands: the decision stage as the paper runs it.

The bf16 models have 8 layers.  The layers of a model are alike, so the time of a layer is what 8 of them show, and at
8 layers the logits of two implementations that add in another order can still be compared: each flipped bf16 rounding
flips more of them downstream, and at 32 layers the logits of the 7B-class model move by 3 % of their size (at 8 by 0.9 %).
For the same reason the bf16 step is timed as its two stages (it equals their composition bit for bit): a draw from
16384 near-uniform entries lands elsewhere when the logits move by a percent.
"""
import math

import torch

import paper_2601_05149_amd as mulo

DEV = "cuda:0"
MODELS = {
    "tiny": dict(n_layers=2, d_model=256, n_heads=4, head_dim=64, d_ffn=688, vocab=1024, dtype="f32"),
    "small": dict(n_layers=8, d_model=1024, n_heads=16, head_dim=64, d_ffn=2816, vocab=8192, dtype="bf16"),
    "7b": dict(n_layers=8, d_model=4096, n_heads=32, head_dim=128, d_ffn=11008, vocab=16384, dtype="bf16"),
}


def listed():
    return [
        # the float32 configuration, its first block: 256 tokens in one step, many small launches
        dict(name="step_f32_256", kind="step", model="tiny", B=1, w=8, h=8, r=2, P=32, radius=1),
        # a block of the small decoder (head dimension 64) in the middle of its image
        dict(name="block_small_4x256", kind="forward", model="small", B=4, L=256, P=576, copy=False, embeds=False),
        # one image at a time: the batch-1 block of the 48 x 48 grid, half of the image committed
        dict(name="block_7b_1x576", kind="forward", model="7b", B=1, L=576, P=1280, copy=False, embeds=False),
        # the high-resolution block, last of its image: the longest cache
        dict(name="block_7b_4x1024", kind="forward", model="7b", B=4, L=1024, P=3200, copy=False, embeds=False),
        # the largest throughput workload: 16384 tokens in one pass
        dict(name="block_7b_16x1024", kind="forward", model="7b", B=16, L=1024, P=3200, copy=False, embeds=False),
        # prefill of a conditioning prefix of ragged length, given as embeddings (guidance doubles the sequences)
        dict(name="prefill_7b_2x93", kind="forward", model="7b", B=2, L=93, P=0, copy=False, embeds=True),
        # one token of one sequence: the lowest latency the library is asked for
        dict(name="token_7b_1", kind="forward", model="7b", B=1, L=1, P=2100, copy=False, embeds=False),
        # one token of four sequences, end of the image, weights kept in streaming order
        dict(name="token_7b_4_copy", kind="forward", model="7b", B=4, L=1, P=4223, copy=True, embeds=False),
        # a re-sampling pass over 13 islands of each of 4 sequences
        dict(name="islands_7b_4x13", kind="islands", model="7b", B=4, L=1024, P=3200, n=13, copy=True),
        # the same for 16 sequences: 160 positions
        dict(name="islands_7b_16x10", kind="islands", model="7b", B=16, L=1024, P=3200, n=10, copy=True),
        # decision stage of the high-resolution block: radius 2, draft = target logits + noise
        dict(name="decide_4x1024", kind="decide", V=16384, B=4, w=32, h=8, r=2, radius=2, sigma=1.0),
        # the paper's setting: guidance of scale 4, pooled threshold rule, re-draws from the target, island labels
        dict(name="guided_2x1024", kind="guided", V=16384, B=2, w=32, h=8, r=2, radius=1, pool=8, tau=1e-4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["block", "block", "block", "token", "prefill", "islands", "decide", "guided", "step"])
    if kind == "step":
        r = rng.choice([2, 4])
        w, h = (rng.randint(4, 12), rng.randint(2, 12)) if r == 2 else (rng.randint(2, 6), rng.randint(1, 6))
        return dict(kind="step", model="tiny", B=rng.randint(1, 4), w=w, h=h, r=r, P=rng.randint(1, 300), radius=rng.randint(0, 3))
    if kind == "block":
        model = rng.choice(["small", "7b", "7b"])
        B, rows, W = rng.choice([1, 1, 2, 3, 4, 8, 16]), rng.randint(2, 32), 2 * rng.randint(6, 16)
        L = min(rows * W, 1024)
        return dict(kind="forward", model=model, B=B, L=L, P=rng.randint(1, 3200), copy=False, embeds=False)
    if kind == "prefill":
        L = _log(rng, 8, 300)
        return dict(kind="forward", model=rng.choice(["small", "7b"]), B=rng.choice([1, 2, 4, 8]), L=L, P=0, copy=False, embeds=rng.random() < 0.5)
    if kind == "token":
        return dict(kind="forward", model=rng.choice(["small", "7b", "7b"]), B=_log(rng, 1, 32), L=1, P=rng.randint(60, 4200), copy=rng.random() < 0.5, embeds=False)
    if kind == "islands":
        return dict(kind="islands", model=rng.choice(["small", "7b"]), B=rng.choice([1, 2, 4, 8, 16]), L=1024, P=rng.randint(60, 3200), n=rng.randint(1, 10), copy=rng.random() < 0.7)
    w, h, r = rng.choice([(8, 8, 2), (16, 8, 2), (24, 6, 2), (32, 8, 2), (16, 4, 4), (11, 5, 3)])
    B, V = rng.choice([1, 2, 4, 7]), rng.choice([1024, 8192, 16384, 16384, 10004, 32768])
    if kind == "decide":
        return dict(kind="decide", V=V, B=B, w=w, h=h, r=r, radius=rng.randint(0, 2), sigma=rng.choice([0.5, 1.0, 2.0]))
    return dict(kind="guided", V=V, B=min(B, 4), w=w, h=h, r=r, radius=rng.randint(0, 3), pool=rng.choice([1, 4, 8, 100]), tau=1.6 / V)


# ---- what a user's program has in hand -------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _weights(m, g):
    nl, d, f, V = m["n_layers"], m["d_model"], m["d_ffn"], m["vocab"]
    dt = torch.bfloat16 if m["dtype"] == "bf16" else torch.float32
    shapes = dict(embed=(V, d), wq=(nl, d, d), wk=(nl, d, d), wv=(nl, d, d), wo=(nl, d, d), w_gate=(nl, f, d),
                  w_up=(nl, f, d), w_down=(nl, d, f), lm_head=(V, d))
    w = {k: torch.empty(s, dtype=dt, device=DEV).normal_(0.0, 0.02, generator=g) for k, s in shapes.items()}
    w.update(attn_norm=torch.ones(nl, d, dtype=dt, device=DEV), ffn_norm=torch.ones(nl, d, dtype=dt, device=DEV),
             final_norm=torch.ones(d, dtype=dt, device=DEV))
    return w


def _rope(max_seq, dh):
    theta = 10000.0 ** (-2.0 * torch.arange(dh // 2, dtype=torch.float64, device=DEV) / dh)
    ang = torch.arange(max_seq, dtype=torch.float64, device=DEV)[:, None] * theta[None, :]
    return ang.cos().float().contiguous(), ang.sin().float().contiguous()


def _model(m, g, B, max_seq, max_block, copy=False):
    """Weights, context and a cache whose rows hold N(0, 1) values (a prefix and committed blocks)."""
    cos, sin = _rope(max_seq, m["head_dim"])
    ctx = mulo.mulo_create(mulo.make_cfg(m, B, max_seq, max_block, stream_copy=copy), _weights(m, g), cos, sin)
    kv = mulo.alloc_kv(ctx, DEV, zero=False)
    for t in kv:
        t.normal_(generator=g)
    return ctx, kv


def _tokens(g, shape, V):
    return torch.randint(0, V, shape, generator=g, device=DEV, dtype=torch.int32)


def _sample(logits, g):
    """One draw per row of softmax(logits)."""
    u = torch.rand(logits.shape, generator=g, device=DEV).clamp_(1e-20, 1.0 - 1e-7)
    return u.log_().neg_().log_().neg_().add_(logits).argmax(-1).to(torch.int32).contiguous()


def _decision_outputs(B, L):
    i32, u8 = torch.int32, torch.uint8
    return dict(tokens_out=torch.empty(B, L, dtype=i32, device=DEV), accept=torch.empty(B, L, dtype=u8, device=DEV),
                mask=torch.empty(B, L, dtype=u8, device=DEV), t0=torch.empty(B, dtype=i32, device=DEV),
                stats=torch.empty(B, 4, dtype=i32, device=DEV))


def _decision_ctx(V, B, L):
    """A context for the decision stage alone: it uses the vocabulary and the workspace only."""
    m = dict(n_layers=1, d_model=128, n_heads=2, head_dim=64, d_ffn=128, vocab=V, dtype="bf16")
    cos, sin = _rope(L + 8, 64)
    return mulo.mulo_create(mulo.make_cfg(m, B, (L + 15) // 8 * 8, (L + 3) // 4 * 4), _weights(m, _gen(0)), cos[:(L + 15) // 8 * 8].contiguous(),
                            sin[:(L + 15) // 8 * 8].contiguous())


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = dict(case=case, seed=seed, out={})
    if kind == "step":
        m = MODELS[case["model"]]
        B, L, V = case["B"], case["w"] * case["h"] * case["r"] ** 2, m["vocab"]
        s["ctx"], s["kv"] = _model(m, g, B, case["P"] + L, L)
        s["draft"] = torch.randn(B, case["h"] * case["w"], V, generator=g, device=DEV).mul_(2.0)
        s["draft_tokens"] = _sample(s["draft"], g)
        s["prev"] = _tokens(g, (B,), V)
        s["out"] = dict(_decision_outputs(B, L), tokens_hi=torch.empty(B, L, dtype=torch.int32, device=DEV),
                        logits=torch.empty(B, L, V, device=DEV))
    elif kind == "forward":
        m = MODELS[case["model"]]
        B, L, V = case["B"], case["L"], m["vocab"]
        s["ctx"], s["kv"] = _model(m, g, B, (case["P"] + L + 7) // 8 * 8, (L + 3) // 4 * 4, case["copy"])
        s["tokens"] = _tokens(g, (B, L), V)
        s["embeds"] = torch.empty(B, L, m["d_model"], dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g) if case["embeds"] else None
        s["logits"] = torch.empty(B, L, V, device=DEV)
    elif kind == "islands":
        m = MODELS[case["model"]]
        B, L, n, V = case["B"], case["L"], case["n"], m["vocab"]
        s["ctx"], s["kv"] = _model(m, g, B, (case["P"] + L + 7) // 8 * 8, L, case["copy"])
        # n marked positions of every sequence, one in each of n stretches of the block and never next to each other:
        # each is an island of its own, of rank 0
        at = (torch.arange(n, device=DEV) * (L // n))[None, :] + torch.randint(2, L // n - 2, (B, n), generator=g, device=DEV)
        s["mask"] = torch.zeros(B, L, dtype=torch.uint8, device=DEV).scatter_(1, at, 1)
        s["rank"] = s["mask"].to(torch.int32) - 1
        s["first"] = _tokens(g, (B, L), V)
        s["tokens"] = s["first"].clone()
        s["prev"] = _tokens(g, (B,), V)
        s["logits"] = torch.zeros(B, L, V, device=DEV)
    else:
        B, V, w, h, r = case["B"], case["V"], case["w"], case["h"], case["r"]
        L = w * h * r * r
        s["nbr"] = None
        child0 = (torch.arange(h, device=DEV)[:, None] * (r * r * w) + torch.arange(w, device=DEV)[None, :] * r).reshape(-1)
        if kind == "decide":
            s["ctx"] = _decision_ctx(V, B, L)
            s["logits"] = torch.randn(B, L, V, generator=g, device=DEV).mul_(1.28)
            s["draft"] = s["logits"][:, child0, :].add(torch.randn(B, h * w, V, generator=g, device=DEV), alpha=case["sigma"])
            s["draft_tokens"] = _sample(s["draft"], g)
            s["hi"] = torch.empty(B, L, dtype=torch.int32, device=DEV)
            s["q_lo"] = torch.empty(B, h * w, V, device=DEV)
            s["q_row"] = torch.empty(L, dtype=torch.int32, device=DEV)
        else:
            s["ctx"] = _decision_ctx(V, 2 * B, L)
            s["logits"] = torch.randn(2 * B, L, V, generator=g, device=DEV).mul_(1.28)     # conditional, then unconditional
            s["logits"][:B].mul_(0.2).add_(s["logits"][B:])
            guided = s["logits"][B:] + 4.0 * (s["logits"][:B] - s["logits"][B:])
            s["hi"] = _sample(guided, g)
            del guided
            if case["pool"] > 1:
                s["nbr"] = _tokens(g, (V, case["pool"]), V)
                s["nbr"][:, 0] = torch.arange(V, device=DEV)
            s["labels"] = [torch.empty(B, L, dtype=torch.int32, device=DEV), torch.empty(B, L, dtype=torch.int32, device=DEV),
                           torch.empty(B, 2, dtype=torch.int32, device=DEV)]
        s["out"] = _decision_outputs(B, L)
    return s


def run(s):
    case, o = s["case"], s["out"]
    kind, B = case["kind"], case["B"]
    if kind == "forward":
        L, P = case["L"], case["P"]
        mulo.mulo_verify_forward(s["ctx"], s["kv"], B, L, P, None if case["embeds"] else s["tokens"], s["embeds"], s["logits"])
        return s["logits"], s["kv"][0][:, :, :, P:P + L], s["kv"][1][:, :, :, :, P:P + L]
    if kind == "islands":
        L, P = case["L"], case["P"]
        s["tokens"].copy_(s["first"])
        mulo.mulo_resample_islands(s["ctx"], s["kv"], B, P, L, 1, case["n"], s["seed"], 3, s["prev"], s["mask"], s["rank"],
                                   s["tokens"], s["logits"])
        return s["tokens"], s["logits"], s["kv"][0][:, :, :, P:P + L], s["kv"][1][:, :, :, :, P:P + L]
    w, h, r = case["w"], case["h"], case["r"]
    W, L = w * r, w * h * r * r
    if kind == "step":
        p = mulo.make_params(h * r, W, 0, L, case["radius"], seed=s["seed"], rng_counter=5)
        mulo.mulo_verify_step(s["ctx"], s["kv"], B, case["P"], p, h, w, r, s["draft"], 0, s["draft_tokens"], s["prev"],
                              o["tokens_out"], o["accept"], o["mask"], o["t0"], o["stats"], o["tokens_hi"], o["logits"])
        return o, s["kv"][0][:, :, :, case["P"]:], s["kv"][1][:, :, :, :, case["P"]:]
    V = case["V"]
    if kind == "decide":
        mulo.mulo_upsample_draft(s["ctx"], B, h, w, r, s["draft"], 0, s["draft_tokens"], s["hi"], s["q_lo"], s["q_row"])
        p = mulo.make_params(h * r, W, 0, L, case["radius"], seed=s["seed"], rng_counter=5)
        mulo.mulo_accept_local_resample(s["ctx"], B, p, s["logits"], s["q_lo"], s["q_row"], h * w * V, s["hi"],
                                        o["tokens_out"], o["accept"], o["mask"], o["t0"], o["stats"])
        return o, s["hi"], s["q_lo"], s["q_row"]
    p = mulo.make_params(h * r, W, 0, L, case["radius"], pool_k=case["pool"], nbr=s["nbr"], resample_mode=2, seed=s["seed"],
                         rng_counter=5, accept_mode=mulo.MULO_ACCEPT_TAU, tau=case["tau"], cfg_scale=4.0)
    mulo.mulo_accept_local_resample(s["ctx"], B, p, s["logits"], None, None, 0, s["hi"], o["tokens_out"], o["accept"],
                                    o["mask"], o["t0"], o["stats"])
    mulo.mulo_rejection_islands(s["ctx"], B, W, 0, L, o["mask"], *s["labels"])
    return o, s["labels"]


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def _forward_work(m, tokens, seqs, keys_read, pairs):
    """tokens in the pass; cache rows read (all sequences); (query, key) pairs attended to."""
    nl, d, f, V = m["n_layers"], m["d_model"], m["d_ffn"], m["vocab"]
    e = 2 if m["dtype"] == "bf16" else 4
    weights = nl * (4 * d * d + 3 * d * f) + V * d
    return dict(bytes=e * (weights + 2 * nl * d * (keys_read + tokens) + tokens * d) + 4 * tokens * V,
                flops=2.0 * tokens * weights + 4.0 * nl * d * pairs)


def work(case):
    kind, B = case["kind"], case["B"]
    if kind == "forward":
        L, P = case["L"], case["P"]
        return _forward_work(MODELS[case["model"]], B * L, B, B * P, B * (L * P + L * (L + 1) / 2))
    if kind == "islands":
        t, keys = B * case["n"], case["P"] + case["L"] / 2
        return _forward_work(MODELS[case["model"]], t, B, B * (case["P"] + case["L"]), t * keys)
    r = case["r"]
    n_lo = case["w"] * case["h"]
    L = n_lo * r * r
    if kind == "step":
        m = MODELS[case["model"]]
        w = _forward_work(m, B * L, B, B * case["P"], B * (L * case["P"] + L * (L + 1) / 2))
        return dict(bytes=w["bytes"] + 4 * m["vocab"] * B * n_lo, flops=w["flops"])
    V = case["V"]
    if kind == "decide":   # logits and draft read once, draft distributions written once
        return dict(bytes=4.0 * V * B * (L + 2 * n_lo), flops=0)
    return dict(bytes=4.0 * V * 2 * B * L, flops=0)


def tolerance(case):
    if case["kind"] in ("forward", "islands"):   # 8 layers of bf16 activations (see above); a marked token may land elsewhere
        return dict(rel=0.03, max=0.5, differ=0.01)
    return dict(rel=1e-5, differ=0.001)           # float32 sums; whole values differ at ties only
