"""GPU parity of the decision stage (up-sampling, accept test, local expansion,
residual re-draw) against the CPU oracle, through the C ABI.

Tolerances: token / mask / index outputs bit-exact; accept flags may differ only
at near ties |pbar - u q| < 1e-4 q (count reported); re-drawn tokens may differ
only when the integer threshold lies within 2^-20 of a CDF boundary;
probabilities within 1e-5 absolute."""
import numpy as np
import pytest
import torch

import paper_2601_05149_amd as mulo
from oracle import step as ST
from oracle import upsample as UP
from tests.gpu_util import DEV, compare_decisions, decide_buffers, dev, make_ctx, say, to_np
from workloads import generators as G

pytestmark = pytest.mark.gpu

_CTX = {}


def decide_ctx(V, max_batch, max_block):
    """A context whose decoder is a stub (the decision entry points only need
    the vocabulary, the stream and the row-statistics workspace)."""
    key = (V, max_batch, max_block)
    if key not in _CTX:
        m = dict(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=64, vocab=V, dtype="f32", rms_eps=1e-5)
        w = G.make_weights(m, seed=0, threads=4)
        _CTX[key] = make_ctx(m, w, max_batch, max_block + 8, max_block)[0]
    return _CTX[key]


def clean_inputs(B, L, V, sigma, seed):
    """Target logits N(0, 1.28) i.i.d., draft logits = target + sigma * noise,
    draft tokens drawn from softmax(draft logits)."""
    zp = G.normal_logits((B, L, V), 1.28, seed, tag=10)
    zq = zp + sigma * G.normal_logits((B, L, V), 1.0, seed, tag=11)
    q = UP.softmax_rows(zq).astype(np.float32)
    toks = G.sample_categorical(zq, seed, tag=12)
    return zp, q, toks


def run_decide(ctx, zp, q, toks, q_row=None, p_probs=False, **pk):
    B, L, V = zp.shape
    nbr = pk.pop("nbr", None)
    nbr_d = dev(nbr) if nbr is not None else None
    params = mulo.make_params(nbr=nbr_d, pool_k=1 if nbr is None else nbr.shape[1], **pk)
    out = decide_buffers(B, L)
    pp = torch.empty(B, L, V, device=DEV) if p_probs else None
    mulo.mulo_accept_local_resample(ctx, B, params, dev(zp, torch.float32),
                                    None if q is None else dev(q, torch.float32),
                                    None if q_row is None else dev(q_row, torch.int32),
                                    0 if q is None else q.shape[1] * V, dev(toks, torch.int32), out["tokens_out"],
                                    out["accept"], out["mask"], out["t0"], out["stats"], pp)
    torch.cuda.synchronize()
    res = to_np(out)
    if pp is not None:
        res["p"] = pp.cpu().numpy()
    return res


# ------------------------------------------------------------------ Step 2
@pytest.mark.parametrize("B,h,w,r,V", [(1, 8, 8, 2, 1024), (2, 5, 7, 2, 1000), (1, 4, 4, 4, 16384),
                                        (2, 3, 3, 1, 2048), (1, 2, 3, 2, 20000), (3, 6, 2, 3, 8192)])
def test_upsample_parity(B, h, w, r, V):
    say("upsample B=%d h=%d w=%d r=%d V=%d" % (B, h, w, r, V))
    ctx = decide_ctx(V, 4, 64)
    dl = G.normal_logits((B, h * w, V), 2.0, seed=1, tag=V)
    dt = G.uniform_tokens((B, h * w), V, seed=1, tag=V)
    x_hi, q_lo, q_row, q_hi = UP.upsample_draft(dl, dt, h, w, r, materialise=True)
    T = h * r * w * r
    g = dict(tokens_hi=torch.empty(B, T, dtype=torch.int32, device=DEV), q_lo=torch.empty(B, h * w, V, device=DEV),
             q_row=torch.empty(T, dtype=torch.int32, device=DEV), q_hi=torch.empty(B, T, V, device=DEV))
    mulo.mulo_upsample_draft(ctx, B, h, w, r, torch.tensor(dl, device=DEV), 0, torch.tensor(dt, device=DEV),
                             g["tokens_hi"], g["q_lo"], g["q_row"], g["q_hi"])
    torch.cuda.synchronize()
    g = to_np(g)
    assert np.array_equal(g["tokens_hi"], x_hi) and np.array_equal(g["q_row"], q_row)
    err = np.abs(g["q_lo"] - q_lo).max()
    say("  max |q_lo - oracle| = %.3g" % err)
    assert err <= 1e-5
    assert np.abs(g["q_lo"].astype(np.float64).sum(-1) - 1).max() < 1e-5
    assert np.array_equal(g["q_hi"], g["q_lo"][:, q_row])           # children carry the parent's row, bit for bit
    # probabilities as input are copied unchanged
    g2 = torch.empty(B, h * w, V, device=DEV)
    mulo.mulo_upsample_draft(ctx, B, h, w, r, torch.tensor(q_lo, device=DEV), 1, torch.tensor(dt, device=DEV),
                             torch.empty(B, T, dtype=torch.int32, device=DEV), g2,
                             torch.empty(T, dtype=torch.int32, device=DEV), None)
    assert np.array_equal(g2.cpu().numpy(), q_lo)


# --------------------------------------------------------------- Steps 4-5 + re-draw
CASES = [
    # B, H, W, n0, L, V, sigma, radius, expand, mode, pool_k
    (1, 16, 16, 0, 256, 1024, 1.0, 1, 1, 0, 1),
    (4, 32, 32, 512, 256, 8192, 1.0, 1, 2, 0, 1),
    (1, 48, 48, 1728, 576, 16384, 1.0, 1, 1, 0, 1),
    (2, 10, 10, 20, 60, 1000, 0.5, 2, 1, 0, 8),        # ragged vocabulary, pooled numerator (Eq. 3)
    (2, 16, 16, 64, 128, 4096, 2.0, 1, 1, 1, 1),       # expanded positions drawn from p
    (2, 16, 16, 0, 256, 2048, 0.5, -1, 1, 0, 1),       # raster-scan rule
    (2, 16, 16, 0, 256, 2048, 1.0, 0, 1, 0, 1),        # radius 0: only the rejected positions
    (1, 8, 8, 0, 64, 20000, 1.0, 3, 1, 0, 1),          # vocabulary beyond the register-resident path
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%d_%dx%d_n%d_L%d_V%d_s%g_r%d_e%d_m%d_k%d" % c)
def test_decide_parity(case):
    B, H, W, n0, L, V, sigma, radius, expand, mode, k = case
    say("decide case %r" % (case,))
    ctx = decide_ctx(V, 4, 1024)
    zp, q, toks = clean_inputs(B, L, V, sigma, seed=3)
    nbr = G.neighbour_table(V, k, seed=3) if k > 1 else None
    kw = dict(W=W, n0=n0, radius=radius, expand=expand, seed=77, rng_counter=(5 << 32) | 9)
    ref = ST.decide(zp, q, None, toks, nbr=nbr, mode=mode, **kw)
    got = run_decide(ctx, zp, q, toks, p_probs=True, H=H, L=L, nbr=nbr, resample_mode=mode, **kw)
    perr = np.abs(got["p"] - ref["p"]).max()
    rep = compare_decisions(got, ref, toks, q, None, mode=mode, label=str(case))
    say("  acc rate %.3f marked %.3f | max|p err| %.3g | %r" % (ref["accept"].mean(), ref["mask"].mean(), perr, rep))
    assert perr <= 1e-5
    assert rep["sequences_checked"] >= 1
    # run-to-run determinism
    again = run_decide(ctx, zp, q, toks, H=H, L=L, nbr=nbr, resample_mode=mode, **kw)
    for name in ("tokens_out", "accept", "mask", "t0", "stats"):
        assert np.array_equal(again[name], got[name])


def test_q_row_indirection_matches_materialised_rows():
    # q given as low-res rows + q_row (what the step uses) == q given per position
    B, h, w, r, V = 2, 4, 8, 2, 4096
    H, W, L = 8, 16, 128
    ctx = decide_ctx(V, 4, 1024)
    dl = G.normal_logits((B, h * w, V), 2.0, seed=4)
    dt = G.sample_categorical(dl, seed=4)
    x_hi, q_lo, q_row, q_hi = UP.upsample_draft(dl, dt, h, w, r, materialise=True)
    zp = q_hi * 0 + np.log(np.maximum(q_hi, 1e-30)) + G.normal_logits((B, L, V), 1.0, seed=4, tag=1)
    kw = dict(W=W, n0=0, radius=1, expand=1, seed=1, rng_counter=2)
    ref = ST.decide(zp, q_lo, q_row, x_hi, **kw)
    a = run_decide(ctx, zp.astype(np.float32), q_lo, x_hi, q_row=q_row, H=H, L=L, **kw)
    b = run_decide(ctx, zp.astype(np.float32), q_hi, x_hi, H=H, L=L, **kw)
    for name in ("tokens_out", "accept", "mask", "t0", "stats"):
        assert np.array_equal(a[name], b[name])
    rep = compare_decisions(a, ref, x_hi, q_lo, q_row, label="q_row")
    say("  q_row case: acc %.3f %r" % (ref["accept"].mean(), rep))


def test_q_equal_p_accepts_everything_on_device():
    B, L, V = 2, 128, 8192
    ctx = decide_ctx(V, 4, 1024)
    zp, _, toks = clean_inputs(B, L, V, 1.0, seed=5)
    first = run_decide(ctx, zp, np.full((B, L, V), 1.0 / V, np.float32), toks, p_probs=True, H=8, W=16, n0=0, L=L,
                       radius=1, seed=0, rng_counter=0)
    got = run_decide(ctx, zp, first["p"], toks, H=8, W=16, n0=0, L=L, radius=1, seed=0, rng_counter=0)
    assert got["accept"].all() and not got["mask"].any()
    assert (got["t0"] == L).all() and np.array_equal(got["tokens_out"], toks)
    assert np.array_equal(got["stats"][:, :3], [[L, 0, 0]] * B)


def test_all_rejected_empty_residual_and_out_of_range_tokens():
    B, L, V = 1, 32, 1024
    ctx = decide_ctx(V, 4, 1024)
    zp = G.normal_logits((B, L, V), 1.0, seed=6)
    zp[:, :, :8] -= 60.0                              # target has (numerically) no mass on the first 8 entries
    q = np.zeros((B, L, V), np.float32)
    q[:, :, :8] = 0.125                               # draft has all of its mass there
    toks = G.uniform_tokens((B, L), 8, seed=6)
    kw = dict(W=8, n0=0, radius=1, expand=1, seed=3, rng_counter=1)
    ref = ST.decide(zp, q, None, toks, **kw)
    got = run_decide(ctx, zp, q, toks, H=4, L=L, **kw)
    assert not ref["accept"].any() and ref["t0"][0] == 0 and ref["mask"].all()
    rep = compare_decisions(got, ref, toks, q, None, label="all rejected")
    assert rep["flips"] == 0
    # q >= p everywhere (q need not be normalised for the test) and a position marked by a rejected
    # neighbour: the residual max(0, p - q) is empty on both sides -> the draw falls back to p
    p = ST.A.target_probs(zp)
    q2 = (p * np.float32(1.001)).astype(np.float32)
    q2[0, 5] = q[0, 5]                                # only position 5 is rejected
    toks2 = toks.copy()
    ref2 = ST.decide(zp, q2, None, toks2, **kw)
    got2 = run_decide(ctx, zp, q2, toks2, H=4, L=L, **kw)
    assert ref2["accept"].sum() >= L - 2 and not ref2["accept"][0, 5] and ref2["mask"].sum() > 1
    compare_decisions(got2, ref2, toks2, q2, None, label="empty residual")
    # ids outside the codebook are clamped, never dereferenced
    bad = toks.copy()
    bad[0, 3], bad[0, 4] = V + 5, -3
    clamped = np.clip(bad, 0, V - 1)
    ref3 = ST.decide(zp, q, None, clamped, **kw)
    got3 = run_decide(ctx, zp, q, bad, H=4, L=L, **kw)
    compare_decisions(got3, ref3, clamped, q, None, label="clamped ids")


def test_argument_errors_are_reported_not_launched():
    ctx = decide_ctx(1024, 4, 1024)
    zp, q, toks = clean_inputs(1, 64, 1024, 1.0, seed=7)
    with pytest.raises(mulo.MuloError) as e:
        run_decide(ctx, zp, q, toks, H=8, W=7, n0=0, L=64, radius=1, seed=0, rng_counter=0)   # L not whole rows
    assert e.value.status == 2
    with pytest.raises(mulo.MuloError) as e:
        run_decide(ctx, zp, q, toks, H=4, W=8, n0=0, L=64, radius=1, seed=0, rng_counter=0)   # block past the grid
    assert e.value.status == 2
    with pytest.raises(mulo.MuloError) as e:
        run_decide(ctx, zp, q, toks, H=8, W=8, n0=0, L=64, radius=-3, seed=0, rng_counter=0)
    assert e.value.status == 3


@pytest.mark.parametrize("name,B,L,radius", [("cfg4", 4, 1024, 2), ("cfg5_L256", 16, 256, 1), ("cfg5_L512", 16, 512, 1),
                                                ("cfg5_L1024", 16, 1024, 1)])
def test_decide_full_size(name, B, L, radius):
    """Decision stage at the full shape of the 7B-class workloads (V = 16384,
    64x64 grid, last block), in the launch configuration the benchmark times."""
    V, H, W = 16384, 64, 64
    say("full-size decide %s" % name)
    ctx = decide_ctx(V, 16, 1024)
    zp, q, toks = clean_inputs(B, L, V, 1.0, seed=8)
    kw = dict(W=W, n0=H * W - L, radius=radius, expand=1, seed=0, rng_counter=3)
    ref = ST.decide(zp, q, None, toks, **kw)
    got = run_decide(ctx, zp, q, toks, H=H, L=L, **kw)
    rep = compare_decisions(got, ref, toks, q, None, label=name)
    say("  %s: acc %.3f marked %.3f %r" % (name, ref["accept"].mean(), ref["mask"].mean(), rep))
    assert rep["sequences_checked"] >= B - 2


# --------------------------------------------------------------- threshold rule (Eq. 5)
TAU_CASES = [
    # B, H, W, n0, L, V, tau, radius, mode, pool_k, with_q
    (2, 16, 16, 0, 256, 1024, 1e-3, 1, 2, 1, False),       # the paper's rule: no draft distribution at all
    (4, 32, 32, 512, 256, 8192, 1e-4, 1, 2, 1, False),
    (1, 48, 48, 1728, 576, 16384, 3e-3, 2, 2, 16, False),  # pooled over 16 codebook neighbours
    (2, 10, 10, 20, 60, 1000, 5e-3, 1, 0, 8, True),        # threshold accept, residual re-draw (needs q)
    (1, 8, 8, 0, 64, 20000, 1e-4, 1, 2, 1, False),         # vocabulary beyond the register-resident path
]


@pytest.mark.parametrize("case", TAU_CASES, ids=lambda c: "B%d_%dx%d_n%d_L%d_V%d_tau%g_r%d_m%d_k%d_q%d" % c)
def test_tau_rule_parity(case):
    B, H, W, n0, L, V, tau, radius, mode, k, with_q = case
    say("tau-rule case %r" % (case,))
    ctx = decide_ctx(V, 4, 1024)
    zp, q, toks = clean_inputs(B, L, V, 1.0, seed=5)
    nbr = G.neighbour_table(V, k, seed=5) if k > 1 else None
    kw = dict(W=W, n0=n0, radius=radius, expand=1, seed=31, rng_counter=(2 << 32) | 4)
    ref = ST.decide(zp, q if with_q else None, None, toks, nbr=nbr, mode=mode, accept_mode=1, tau=tau, **kw)
    got = run_decide(ctx, zp, q if with_q else None, toks, p_probs=True, H=H, L=L, nbr=nbr, resample_mode=mode,
                     accept_mode=mulo.MULO_ACCEPT_TAU, tau=tau, **kw)
    rep = compare_decisions(got, ref, toks, q, None, mode=mode, label=str(case))
    say("  acc rate %.3f marked %.3f | %r" % (ref["accept"].mean(), ref["mask"].mean(), rep))
    assert 0.02 < ref["accept"].mean() < 0.999          # the case exercises both outcomes
    assert np.abs(got["p"] - ref["p"]).max() <= 1e-5
    assert rep["sequences_checked"] >= 1
    # no random number enters the accept decision: another counter gives the same flags and mask
    kw2 = dict(kw, rng_counter=99)
    got2 = run_decide(ctx, zp, q if with_q else None, toks, H=H, L=L, nbr=nbr, resample_mode=mode,
                      accept_mode=mulo.MULO_ACCEPT_TAU, tau=tau, **kw2)
    assert np.array_equal(got2["accept"], got["accept"]) and np.array_equal(got2["mask"], got["mask"])


def test_tau_rule_limits_and_errors_on_device():
    B, H, W, L, V = 2, 8, 8, 64, 512
    ctx = decide_ctx(V, 4, 1024)
    zp, q, toks = clean_inputs(B, L, V, 1.0, seed=6)
    kw = dict(H=H, W=W, n0=0, L=L, radius=1, resample_mode=2, accept_mode=mulo.MULO_ACCEPT_TAU)
    allacc = run_decide(ctx, zp, None, toks, tau=0.0, **kw)
    assert allacc["accept"].all() and not allacc["mask"].any() and np.array_equal(allacc["tokens_out"], toks)
    none = run_decide(ctx, zp, None, toks, tau=1.5, **kw)
    assert not none["accept"].any() and none["mask"].all() and (none["t0"] == 0).all()
    # a missing draft distribution is an error wherever it would be read
    for bad in (dict(kw, resample_mode=0), dict(kw, accept_mode=mulo.MULO_ACCEPT_RATIO)):
        with pytest.raises(mulo.MuloError) as e:
            run_decide(ctx, zp, None, toks, tau=1e-3, **bad)
        assert e.value.status == 1


def test_sampler_words_equal_the_oracle_generator_on_2_pow_20_counters():
    """Uniform target distribution over V = 2^16 entries, everything rejected (threshold above 1) and re-drawn
    from p: the integer inverse CDF then returns the top 16 bits of each position's Philox word, so the
    device generator (counter layout, key schedule, rounds) is compared with the oracle's on 2^20 counters."""
    from oracle import philox as PH
    from oracle import resample as RS
    B, L, V = 4, 1024, 65536
    ctx = decide_ctx(V, B, L)
    z = torch.zeros(B, L, V, device=DEV)
    toks = torch.zeros(B, L, dtype=torch.int32, device=DEV)
    out = decide_buffers(B, L)
    # closed form of the draw for equal weights, checked against the oracle's sampler on a few words
    Wi = RS.integer_weights(np.full(V, 1.0 / V, np.float32))
    for wd in (0, 1, 65535, 65536, 0x7FFFFFFF, 0x80000000, 0xFFFFFFFF, 0x12345678):
        assert RS.draw(Wi, wd) == wd >> 16
    seed = 0x9E3779B97F4A7C15
    n_bad = 0
    for c in range(256):
        ctr = (c << 40) | (c * 2654435761 % (1 << 32))          # low and high counter words both vary
        params = mulo.make_params(32, 32, 0, L, 1, 1, resample_mode=2, seed=seed, rng_counter=ctr,
                                  accept_mode=mulo.MULO_ACCEPT_TAU, tau=1.5)
        mulo.mulo_accept_local_resample(ctx, B, params, z, None, None, 0, toks, out["tokens_out"], out["accept"],
                                        out["mask"], out["t0"], out["stats"], None)
        got = out["tokens_out"].cpu().numpy()
        words = PH.step_words(seed, ctr, PH.STREAM_SAMPLE, B, L)
        n_bad += int((got != (words >> 16).astype(np.int64)).sum())
    say("  sampler words: %d of %d positions differ" % (n_bad, 256 * B * L))
    assert n_bad == 0


# --------------------------------------------------------------- classifier-free guidance
@pytest.mark.parametrize("B,V,scale,amode", [(2, 1024, 4.0, 1), (1, 16384, 4.0, 0), (2, 20000, 1.5, 1), (2, 2048, 1.0, 0)])
def test_guided_decide_parity(B, V, scale, amode):
    say("guided decide B=%d V=%d s=%g accept_mode=%d" % (B, V, scale, amode))
    H, W, L = 8, 8, 64
    ctx = decide_ctx(V, 4, 1024)
    zc, q, toks = clean_inputs(B, L, V, 1.0, seed=8)
    zu = 0.7 * zc + 0.5 * G.normal_logits((B, L, V), 1.0, 8, tag=99)       # correlated with the conditional logits
    kw = dict(W=W, n0=0, radius=1, expand=1, seed=13, rng_counter=21)
    mode = 2 if amode == 1 else 0
    ref = ST.decide(zc, q, None, toks, mode=mode, accept_mode=amode, tau=2e-3, logits_uncond=zu, cfg_scale=scale, **kw)
    z2 = np.ascontiguousarray(np.concatenate([zc, zu], axis=0))           # [2B, L, V]: conditional, then unconditional
    params = mulo.make_params(H, W, 0, L, 1, 1, resample_mode=mode, seed=13, rng_counter=21, accept_mode=amode, tau=2e-3,
                              cfg_scale=scale)
    out = decide_buffers(B, L)
    pp = torch.empty(B, L, V, device=DEV)
    mulo.mulo_accept_local_resample(ctx, B, params, dev(z2, torch.float32), dev(q, torch.float32), None, L * V,
                                    dev(toks, torch.int32), out["tokens_out"], out["accept"], out["mask"], out["t0"],
                                    out["stats"], pp)
    torch.cuda.synchronize()
    got = to_np(out)
    got["p"] = pp.cpu().numpy()
    perr = np.abs(got["p"] - ref["p"]).max()
    rep = compare_decisions(got, ref, toks, q, None, mode=mode, label="guided")
    say("  acc rate %.3f marked %.3f | max|p err| %.3g | %r" % (ref["accept"].mean(), ref["mask"].mean(), perr, rep))
    assert perr <= 1e-5 and rep["sequences_checked"] >= 1
    if scale == 1.0:      # s = 1 is the conditional distribution: same decisions as without guidance
        plain = run_decide(ctx, zc, q, toks, H=H, L=L, resample_mode=mode, accept_mode=amode, tau=2e-3, **kw)
        assert np.array_equal(plain["accept"], got["accept"]) and np.array_equal(plain["tokens_out"], got["tokens_out"])
    with pytest.raises(mulo.MuloError):        # 2 B sequences must fit the context
        mulo.mulo_accept_local_resample(ctx, 3, params, dev(z2, torch.float32), dev(q, torch.float32), None, L * V,
                                        dev(toks, torch.int32), out["tokens_out"], out["accept"], out["mask"], out["t0"],
                                        out["stats"], None)


# ------------------------------------------- the draw from the chunk sums that the accept test leaves
@pytest.mark.parametrize("V", [4, 260, 508, 516, 1028, 2048, 2052, 4096, 8196, 10004, 12288, 12292, 16384, 16388])
@pytest.mark.parametrize("kw", [dict(radius=1), dict(radius=-1, resample_mode=1), dict(radius=0, resample_mode=2),
                                dict(radius=2, resample_mode=1, pool=5), dict(radius=1, cfg_scale=3.0), dict(radius=0),
                                dict(radius=1, accept_mode=1, tau=1e-3, resample_mode=2, cfg_scale=2.0),
                                dict(radius=1, noise=0.1), dict(radius=2, resample_mode=1, noise=0.1)])
def test_draw_from_chunk_sums_equals_the_draw_from_the_rows(V, kw):
    """A bf16 context has room for the chunk sums, so its accept test leaves them for the draw where Eq. 1 is tested without
    pooling, residual weights are drawn from and the radius is not 0 (vocabularies up to 16384); the entry point without a
    context reads each marked row again, and so does the context in the other settings.  All outputs are the same bits:
    vocabularies at the edges of a chunk, of a lane's run of 8 and of the registers, drafts far from the target and close to
    it (few rejected, many positions not marked), and in the residual settings rows whose draft distribution IS the
    target's (an empty residual, re-drawn from p)."""
    kw = dict(kw)
    B, W, rows = 3, 8, 7
    L, pool, noise = W * rows, kw.pop("pool", 1), kw.pop("noise", 0.7)
    key = ("sums", V)
    if key not in _CTX:
        m = dict(n_layers=1, d_model=128, n_heads=2, head_dim=64, d_ffn=128, vocab=V, dtype="bf16", rms_eps=1e-5)
        _CTX[key] = make_ctx(m, G.make_weights(m, seed=0), 2 * B, L + 8, L)[0]
    ctx = _CTX[key]
    g = torch.Generator(device=DEV).manual_seed(V + len(str(kw)))
    guided = kw.get("cfg_scale", 0.0) > 0
    z = torch.randn((2 if guided else 1) * B, L, V, generator=g, device=DEV).mul_(1.5)
    q = torch.softmax(z[:B] + noise * torch.randn(B, L, V, generator=g, device=DEV), dim=-1).contiguous()
    toks = torch.randint(0, V, (B, L), generator=g, device=DEV, dtype=torch.int32)
    toks[:, ::2] = q.argmax(-1)[:, ::2].to(torch.int32)      # where the draft is surest the target is less so: rejections
    pp = torch.empty(B, L, V, device=DEV)
    nbr = None
    if pool > 1:
        pool = min(pool, V)
        nbr = torch.randint(0, V, (V, pool), generator=g, device=DEV, dtype=torch.int32)
        nbr[:, 0] = torch.arange(V, device=DEV)
    params = mulo.make_params(rows, W, 0, L, kw.pop("radius"), pool_k=pool, nbr=nbr, seed=7, rng_counter=3, **kw)
    call = lambda f, *head: (lambda o: (f(*head, B, params, z, q, None, L * V, toks, o["tokens_out"], o["accept"], o["mask"],
                                          o["t0"], o["stats"]), o)[1])(decide_buffers(B, L))
    # every third row of the draft becomes the target distribution itself, as the library computes it
    o = decide_buffers(B, L)
    mulo.mulo_accept_local_resample_static(V, B, params, z, q, None, L * V, toks, o["tokens_out"], o["accept"], o["mask"],
                                           o["t0"], o["stats"], pp)
    q[:, ::3] = pp[:, ::3]
    a = call(mulo.mulo_accept_local_resample, ctx)
    b = call(lambda *x: mulo.mulo_accept_local_resample_static(V, *x))
    torch.cuda.synchronize()
    for k in a:
        assert torch.equal(a[k], b[k]), (V, kw, k, int((a[k] != b[k]).sum()))
    assert V == 4 or int(a["stats"][:, 2].sum()) > 0      # four entries, five of them pooled: nothing is rejected
    assert (a["tokens_out"] >= 0).all() and (a["tokens_out"] < V).all()


# --------------------------------------------------------------- rejection islands (Eq. 8)
def _check_mask_and_counters(dtype, B, W, rows, rho, row0=0):
    """Few and late rejections, so that windows hold rejections in front of, behind and at the position, and sequences that accept
    everything.  t0, mask and counters from the flags by numpy, and every unmarked token kept."""
    L, V = W * rows, 8
    key = (dtype, V, B, L)
    if key not in _CTX:
        m = dict(n_layers=1, d_model=128, n_heads=2, head_dim=64, d_ffn=128, vocab=V, dtype=dtype, rms_eps=1e-5)
        block = (L + 3) // 4 * 4
        _CTX[key] = make_ctx(m, G.make_weights(m, seed=0, threads=4), B, (block + 7) // 8 * 8 + 8, block)[0]
    ctx = _CTX[key]
    rng = np.random.default_rng(7)
    zp = np.zeros((B, L, V), np.float32)
    q = np.full((B, L, V), 1.0 / V, np.float32)
    toks = rng.integers(0, V, (B, L)).astype(np.int32)
    at = [sorted({L // 3, min(L // 3 + 7, L - 1), L - 1}), [L - 2], []]
    for b in range(B):
        zp[b, at[b % 3], toks[b, at[b % 3]]] = -40.0                    # p of the draft token is 0: rejected whatever the uniform
    res = run_decide(ctx, zp, q, toks, H=rows + row0, W=W, n0=row0 * W, L=L, radius=rho, seed=3, rng_counter=1)
    for b in range(B):
        rej = np.flatnonzero(res["accept"][b] == 0)
        t0 = int(rej[0]) if rej.size else L
        assert list(rej) == at[b % 3] and res["t0"][b] == t0
        ii, jj = np.arange(L) // W, np.arange(L) % W
        hit = np.zeros(L, bool) if rho >= 0 else np.full(L, rej.size > 0)
        for t in rej if rho >= 0 else ():
            hit |= np.maximum(abs(ii - t // W), abs(jj - t % W)) <= rho
        want = hit & (np.arange(L) >= t0)
        assert np.array_equal(res["mask"][b] != 0, want)
        assert list(res["stats"][b][:3]) == [L - rej.size, rej.size, int(want.sum())]
        assert np.array_equal(res["tokens_out"][b][~want], toks[b][~want])


@pytest.mark.parametrize("W,rows", [(64, 64), (64, 65), (4097, 1), (1, 4096), (61, 67)])
@pytest.mark.parametrize("rho", [-1, 0, 2, 70])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])   # a bf16 context draws from chunk sums where there is a window (k_sample_sums)
def test_mask_and_counters_of_long_blocks(W, rows, rho, dtype):
    """Three blocks of 4096 positions and a few more, which a launch in front of the re-draw finishes."""
    _check_mask_and_counters(dtype, 3, W, rows, rho)


@pytest.mark.parametrize("B,W,rows,rhos", [
    (1, 64, 64, (-1, 0, 1, 5, 70)), (1, 241, 17, (-1, 0, 5)),   # 4096 positions: the re-draw finishes them; 4097: a launch does
    (4, 64, 16, (-1, 0, 2, 3)), (5, 64, 16, (-1, 0, 2)),        # of several sequences: a launch from 4097 on where it draws from the rows,
    (16, 64, 16, (1, 8)), (17, 61, 16, (1, 8)),                 # from 16385 on where it draws from chunk sums
    (2, 16, 32, (3, 4, 6)), (1, 64, 32, (1, 2, 9)),             # windows within eight flags a row, more, and of more than 256 flags
    (3, 257, 1, (2, 70)), (3, 1, 300, (2, 70)),                 # one row, one column
    (17, 7, 9, (-1, 0, 2, 70)), (1, 1, 5, (0, 3)),              # more sequences than two rounds of eight workgroups; a handful of positions
])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_mask_and_counters_on_both_sides_of_the_rule(B, W, rows, rhos, dtype):
    """Decisions whose re-draw makes mask and counters itself, and the next larger ones, which a launch in front of it finishes; also of a
    block that does not begin the grid."""
    for rho in rhos:
        for row0 in (0, 3):
            _check_mask_and_counters(dtype, B, W, rows, rho, row0)


def _islands_gpu(ctx, mask, W, n0):
    B, L = mask.shape
    isl = torch.empty(B, L, dtype=torch.int32, device=DEV)
    rk = torch.empty(B, L, dtype=torch.int32, device=DEV)
    cnt = torch.empty(B, 2, dtype=torch.int32, device=DEV)
    mulo.mulo_rejection_islands(ctx, B, W, n0, L, dev(mask.astype(np.uint8), torch.uint8), isl, rk, cnt)
    torch.cuda.synchronize()
    return isl.cpu().numpy(), rk.cpu().numpy(), cnt.cpu().numpy()


def test_rejection_islands_parity():
    from oracle import local as LOC
    ctx = decide_ctx(1024, 4, 1024)
    rng = np.random.default_rng(12)
    cases = [(8, 0, 8, 0.3), (16, 4, 8, 0.2), (7, 3, 5, 0.5), (64, 48, 16, 0.12), (64, 0, 64, 0.25), (9, 0, 5, 0.95), (48, 36, 12, 0.0)]
    for W, row0, rows, dens in cases:
        L, n0 = rows * W, row0 * W
        mask = rng.random((3, L)) < dens
        # a serpentine path: the slowest case for label propagation (one island that winds through every other row)
        snake = np.zeros((rows, W), bool)
        snake[::2] = True
        for r in range(1, rows, 2):
            snake[r, W - 1 if (r // 2) % 2 == 0 else 0] = True
        mask[2] = snake.reshape(-1)
        isl, rk, cnt = _islands_gpu(ctx, mask, W, n0)
        for b in range(3):
            ri, rr, n, largest = LOC.rejection_islands(mask[b], W, n0)
            assert np.array_equal(isl[b], ri) and np.array_equal(rk[b], rr), (W, row0, rows, dens, b)
            assert cnt[b].tolist() == [n, largest]
        say("  islands W=%d rows=%d density %.2f: %s islands, largest %s" % (W, rows, dens, cnt[:, 0].tolist(), cnt[:, 1].tolist()))
    with pytest.raises(mulo.MuloError):
        _islands_gpu(ctx, np.zeros((1, 30), bool), 8, 0)       # not whole rows
    with pytest.raises(mulo.MuloError):
        _islands_gpu(ctx, np.zeros((1, 32), bool), 8, 4)       # block does not start on a row


@pytest.mark.parametrize("W,rows", [(64, 256), (128, 64), (61, 51), (1, 130), (130, 1), (3, 1)])
def test_rejection_islands_at_the_sizes_of_the_counters(W, rows):
    """The largest block (one set of member counters in LDS), half of it, an odd one whose segments end inside a row, and
    grids of one column or one row, each sparse, dense, full, a checkerboard (one island by its diagonals), a spiral, empty,
    and with one position marked, the last."""
    from oracle import local as LOC
    L = W * rows
    ctx = decide_ctx(1024, 4, 1024)
    rng = np.random.default_rng(W * 1000 + rows)
    i, j = np.divmod(np.arange(L), W)
    spiral = np.zeros((rows, W), bool)
    r0, r1, c0, c1 = 0, rows, 0, W
    while r1 - r0 > 2 and c1 - c0 > 2:               # rings two apart, joined by one cell each
        spiral[r0, c0:c1] = spiral[r1 - 1, c0:c1] = spiral[r0:r1, c0] = spiral[r0:r1, c1 - 1] = True
        spiral[r0 + 1, c0] = False
        spiral[r0 + 2 if r0 + 2 < rows else r0, min(c0 + 1, W - 1)] = True
        r0, r1, c0, c1 = r0 + 2, r1 - 2, c0 + 2, c1 - 2
    mask = np.stack([rng.random(L) < 0.1, rng.random(L) < 0.45, np.ones(L, bool), (i + j) % 2 == 0, spiral.reshape(-1),
                     np.zeros(L, bool), np.arange(L) == L - 1])
    isl, rk, cnt = _islands_gpu(ctx, mask, W, 0)
    for b in range(len(mask)):
        ri, rr, n, largest = LOC.rejection_islands(mask[b], W, 0)
        assert np.array_equal(isl[b], ri) and np.array_equal(rk[b], rr) and cnt[b].tolist() == [n, largest], (W, rows, b)


def test_rejection_islands_of_a_decided_block():
    """Islands of the mask that the decision stage produced (radius-1 neighbourhoods of scattered rejections)."""
    from oracle import local as LOC
    B, H, W, L, V = 2, 32, 32, 1024, 1024
    ctx = decide_ctx(V, 4, 1024)
    zp, q, toks = clean_inputs(B, L, V, 0.35, seed=4)
    # the paper's threshold rule with a low threshold: a few scattered rejections
    got = run_decide(ctx, zp, None, toks, H=H, W=W, n0=0, L=L, radius=1, expand=1, seed=1, rng_counter=2,
                     resample_mode=2, accept_mode=mulo.MULO_ACCEPT_TAU, tau=1e-4)
    isl, rk, cnt = _islands_gpu(ctx, got["mask"].astype(bool), W, 0)
    for b in range(B):
        ri, rr, n, largest = LOC.rejection_islands(got["mask"][b], W, 0)
        assert np.array_equal(isl[b], ri) and np.array_equal(rk[b], rr) and cnt[b].tolist() == [n, largest]
    say("  decided block: marked %.3f, islands %s, passes %s (sequential would need %s)" % (
        got["mask"].mean(), cnt[:, 0].tolist(), cnt[:, 1].tolist(), got["mask"].sum(1).tolist()))
    assert (cnt[:, 0] > 1).all() and (cnt[:, 1] < got["mask"].sum(1)).all()
